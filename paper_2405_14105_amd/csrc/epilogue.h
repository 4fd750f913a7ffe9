// Fused GEMM epilogues on MFMA output fragments, shared by the window GEMMs
// (gemm.hip) and the prefill GEMM (prefill.hip).
#pragma once

#include "device_util.h"

namespace dsi {

// Inputs of the one epilogue item a thread owns: EPI_RESID the residual and
// gain values, EPI_QKV the rotary (cos, sin) pairs of the item's two feature
// pairs and the cache slot of its row.
struct EpiIn {
  float4 x, g;
  float4 rope;
  int win, pos;   // EPI_QKV: window and cache slot of the row (pos < 0: not cached)
};

// EPI_QKV inputs of row m, n-block nb, features r0..r0+3 of it
__device__ __forceinline__ EpiIn qkv_inputs(const EpiArgs& e, int nb, int r0, int m) {
  EpiIn r{};
  const int bph = e.hd >> 4, nq = e.n_heads * bph, nk = e.n_kv * bph;
  r.win = e.rows.window0 + m / e.rows.rows_per_window;
  r.pos = row_slot(e.rows, m);
  if (nb < nq + nk) {
    const int sb = nb < nq ? nb : nb - nq;
    const int ja = (sb % bph) * 8 + (r0 >> 2) * 2;
    const float2 ca = e.rope[(size_t)m * (e.hd >> 1) + ja];
    const float2 cb = e.rope[(size_t)m * (e.hd >> 1) + ja + 1];
    r.rope = float4{ca.x, ca.y, cb.x, cb.y};
  }
  return r;
}

// Returns the sum of the squared residual values it wrote (EPI_RESID), else 0.
template <int WT, int EPI>
__device__ __forceinline__ float epilogue(const EpiArgs& e, int nb, int r0, int m, int split, f32x4 s,
                                          const EpiIn& pre) {
  switch (EPI) {
    case EPI_STORE: {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = nb * 16 + r0 + j;
        if (n < e.n_valid) e.out[(size_t)m * e.ld + n] = s[j];
      }
      break;
    }
    case EPI_PARTRES: {
      // device-scope stores: written through to the point where the
      // group's last workgroup reads them (no L2 write-back needed)
      float* o = e.out + split * e.part_stride + (size_t)m * e.ld;
      const int n0 = nb * 16 + r0;
      if (n0 + 3 < e.n_valid) {
        store4_device(o + n0, s);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (n0 + j < e.n_valid) __hip_atomic_store(o + n0 + j, s[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      break;
    }
    case EPI_PART: {
      float* o = e.out + split * e.part_stride + (size_t)m * e.ld;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = nb * 16 + r0 + j;
        if (n < e.n_valid) o[n] = s[j];
      }
      break;
    }
    case EPI_SILU: {
      // rows 4g+0, 4g+1: gate of features f, f+1; rows 4g+2, 4g+3: up
      const int f = nb * 8 + (r0 >> 2) * 2;
      if (f + 1 < e.ff) pack_store2(e.pack, WT, m, f, silu_f(s[0]) * s[2], silu_f(s[1]) * s[3]);
      else if (f < e.ff) pack_store(e.pack, WT, m, f, silu_f(s[0]) * s[2]);
      break;
    }
    case EPI_QKV: {
      const int hd = e.hd;
      const int bph = hd >> 4;                       // 16-row blocks per head
      const int nq = e.n_heads * bph, nk = e.n_kv * bph;
      const int win = pre.win, pos = pre.pos;
      if (nb < nq + nk) {
        const int sb = nb < nq ? nb : nb - nq;
        const int h = sb / bph;
        const int ja = (sb % bph) * 8 + (r0 >> 2) * 2;   // pair indices ja, ja+1
        const int half = hd >> 1;
        const float2 ca{pre.rope.x, pre.rope.y};   // rope[m][ja], rope[m][ja + 1]
        const float2 cb{pre.rope.z, pre.rope.w};
        const float a1 = s[0] * ca.x - s[2] * ca.y, a2 = s[2] * ca.x + s[0] * ca.y;
        const float b1 = s[1] * cb.x - s[3] * cb.y, b2 = s[3] * cb.x + s[1] * cb.y;
        if (nb < nq) {
          float* qr = e.q_out + (size_t)m * (e.n_heads * hd) + h * hd;
          qr[ja] = a1;
          qr[ja + half] = a2;
          qr[ja + 1] = b1;
          qr[ja + 1 + half] = b2;
        } else if (pos >= 0) {
          const size_t base = ((size_t)win * e.n_kv + h) * e.maxlen * hd;
          const size_t i0 = base + kc_off(pos, ja, hd), i1 = base + kc_off(pos, ja + half, hd);
          const size_t i2 = base + kc_off(pos, ja + 1, hd), i3 = base + kc_off(pos, ja + 1 + half, hd);
          if (e.kv_bf16) {
            uint16_t* kc = (uint16_t*)e.kcache;
            kc[i0] = f2bf_bits(a1);
            kc[i1] = f2bf_bits(a2);
            kc[i2] = f2bf_bits(b1);
            kc[i3] = f2bf_bits(b2);
          } else {
            float* kc = (float*)e.kcache;
            kc[i0] = a1;
            kc[i1] = a2;
            kc[i2] = b1;
            kc[i3] = b2;
          }
        }
      } else if (pos >= 0) {
        const int vb = nb - nq - nk;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = vb * 16 + r0 + j;
          const int h = n / hd, dd = n % hd;
          const size_t idx = ((size_t)win * e.n_kv + h) * e.maxlen * hd + vc_off(pos, dd, hd);
          if (e.kv_bf16) ((uint16_t*)e.vcache)[idx] = f2bf_bits(s[j]);
          else ((float*)e.vcache)[idx] = s[j];
        }
      }
      break;
    }
    case EPI_RESID: {
      // four consecutive features n0..n0+3 of row m (x, gain prefetched)
      const int n0 = nb * 16 + r0;
      const float xn[4] = {pre.x.x + s[0], pre.x.y + s[1], pre.x.z + s[2], pre.x.w + s[3]};
      *(float4*)(e.x + (size_t)m * e.ld + n0) = float4{xn[0], xn[1], xn[2], xn[3]};
      const float y[4] = {xn[0] * pre.g.x, xn[1] * pre.g.y, xn[2] * pre.g.z, xn[3] * pre.g.w};
      pack_store4(e.pack, WT, m, n0, y);
      return xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3];
    }
  }
  return 0.f;
}

}  // namespace dsi
