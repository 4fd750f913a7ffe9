// Prefill: the layer GEMMs and the attention of up to kWideRows prompt rows
// per forward.
//
// A verification window is bound by streaming the weights once; a prompt of
// hundreds of rows is bound by the matrix cores, if the weights are read once
// for all of them.  In forwards of 64 rows the weights were read n / 64 times:
// 2048 tokens through one 8B layer took 5.1 ms (gate/up 2.00, down 1.24, QKV
// 0.85, O 0.65, attention 0.4); in one forward they take 1.6 ms (gate/up 0.76,
// O and down 0.48 together, QKV 0.21, attention 0.08, the residual and norm
// passes 0.09).
//
// GEMM (bf16 weights).  Same products as the window GEMMs: pre-tiled weights
// against the hi/lo activation packs, two 16x16x32 MFMAs per product, fp32
// sums.  A workgroup of 8 waves makes a tile of NWN * 64 features x MT * 16 rows:
//  * NWN (2, 4 or 8) waves lie along the features, four n-blocks each, and 8 /
//    NWN groups of them split the tile's k-blocks, so two waves share each
//    SIMD whatever the tile; the groups' sums meet in LDS at the end, in group
//    order.
//  * Weight fragments belong to one wave and go from memory to its registers,
//    two k-blocks ahead.  Activation fragments are used by all NWN waves of a
//    group and go through LDS (double buffered, one barrier per k-block):
//    each fragment read there feeds four MFMAs, 64 of LDS's 128 bytes a
//    cycle at full MFMA rate.  Both are stored in fragment order, so every
//    load is 1 KB contiguous and no LDS access conflicts.
//  * A wave's running sum goes into a second set of accumulators every
//    kWideRun k-blocks.  In one chain over all of a wave's k-blocks (up to
//    224 at the 8B shape) the error against 64 bits was 0.9 % larger than in
//    the window kernels, whose waves sum 14-20 (700 rows, d = 4096, fp32
//    cache: 2.482e-6 against 2.461e-6; now 2.458e-6).  The second set is why
//    a tile has at most five row blocks (totals of the fifth and fourth in LDS
//    where the registers are full).  Tiles of 8 x 4 blocks a wave and two
//    waves' K groups, which it replaces, were 1-4 % faster: 2048 rows of four
//    8B layers 5.20 ms, now 5.30; 1000 rows 2.84 and 2.88; 509 rows of eight
//    1B layers 1.28 and 1.30.
//  * K-blocks past the split are zeroed on their way into LDS.
// At the 8B shape and 2048 rows it executes 1.2-1.3 PFLOP/s, the rate of a
// large bf16 library product on the card (1.29).

#include <algorithm>

#include "epilogue.h"

namespace dsi {

namespace {

constexpr int kWideWaves = 8;
constexpr int kWideNb = 4;     // n-blocks per wave
constexpr int kWideRun = 9;    // k-blocks a wave adds up before they go into its total (a multiple of 3)

// Workgroup order: XCD x (ids congruent to x mod 8) takes a contiguous run of
// the tiles, row tiles fastest within groups of eight, so the 32 workgroups
// of an XCD share a few weight and activation tiles through its L2.
struct WideGrid {
  int nt, mtiles;       // tiles along the features and the rows
  int tiles;            // of one K split
  int per_xcd;          // workgroups (tiles of all splits) of one XCD
};

// NT: the weights are read by one row tile only, and loaded nontemporally
template <int MT, int NWN, int EPI, int NT>
__global__ __launch_bounds__(kWideWaves * 64) void k_gemm_wide(GemmArgs a, WideGrid gr) {
  constexpr int KG = kWideWaves / NWN;          // K groups
  constexpr int XT = 2 * MT;                    // activation tiles of a k-block (hi, lo)
  constexpr int XP = (XT + NWN - 1) / NWN;      // of them, copied by one wave
  constexpr int XS = KG * 2 * XT * 64;
  constexpr int RS = kWideWaves * 2 * MT * 64;
  constexpr int TR = MT < 5 || NWN == 8 ? MT : 3;   // row blocks whose totals are in registers
  __shared__ u32x4 sm[XS > RS ? XS : RS];
  __shared__ f32x4 tot_sh[MT > TR ? kWideWaves * kWideNb * (MT - TR) * 64 : 1];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = w % NWN, kg = w / NWN;
  const int t0 = (blockIdx.x & 7) * gr.per_xcd + (blockIdx.x >> 3);
  if (t0 >= gr.tiles * a.S) return;
  const int split = t0 / gr.tiles, tile = t0 - split * gr.tiles;
  constexpr int GM = 8;
  const int mg = tile / (GM * gr.nt), in = tile - mg * (GM * gr.nt);
  const int gm = min(GM, gr.mtiles - mg * GM);
  const int nti = in / gm, mti = mg * GM + in % gm;
  const int Mb = (a.M + 15) >> 4;
  const int mb0 = mti * MT;
  const int nb0 = (nti * NWN + wn) * kWideNb;
  const int k0 = (split * a.Kb) / a.S, k1 = ((split + 1) * a.Kb) / a.S;
  const int n = (k1 - k0 + KG - 1) / KG;

  const u32x4* __restrict__ W = (const u32x4*)a.W;
  const u32x4* __restrict__ Xh = (const u32x4*)a.Xhi;
  const u32x4* __restrict__ Xl = (const u32x4*)a.Xlo;
  size_t tb[kWideNb];
  int ts[kWideNb];
#pragma unroll
  for (int j = 0; j < kWideNb; ++j) {
    const int nb = min(nb0 + j, a.Nb - 1), gi = nb / a.G;
    tb[j] = (size_t)gi * a.G * a.Kb + (nb - gi * a.G);
    ts[j] = min(a.G, a.Nb - gi * a.G);
  }
  auto load_w = [&](u32x4 (&d)[kWideNb], int i) {
    const int kb = min(k0 + i * KG + kg, k1 - 1);
#pragma unroll
    for (int j = 0; j < kWideNb; ++j) {
      const u32x4* p = &W[(tb[j] + (size_t)kb * ts[j]) * 64 + lane];
      d[j] = NT ? __builtin_nontemporal_load(p) : *p;
    }
  };
  auto load_x = [&](u32x4 (&d)[XP], int i) {
    const int kb = min(k0 + i * KG + kg, k1 - 1);
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      const int t = min(wn + NWN * p, XT - 1);
      const int mb = min(mb0 + (t >> 1), Mb - 1);
      d[p] = ((t & 1) ? Xl : Xh)[((size_t)mb * a.Kb + kb) * 64 + lane];
    }
  };
  u32x4* const xs = sm + kg * 2 * XT * 64;
  f32x4* const tot_l = tot_sh + (MT > TR ? w * kWideNb * (MT - TR) * 64 + lane : 0);
  // k-blocks past the split are multiplied as zeros (the loop runs whole
  // steps of KG k-blocks, three at a time)
  auto store_x = [&](const u32x4 (&d)[XP], int i) {
    const uint32_t keep = k0 + i * KG + kg < k1 ? ~0u : 0u;
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      const int t = wn + NWN * p;
      if (XT % NWN == 0 || t < XT) xs[((i & 1) * XT + t) * 64 + lane] = d[p] & keep;
    }
  };
  auto sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  f32x4 acc[kWideNb][MT];
#pragma unroll
  for (int j = 0; j < kWideNb; ++j)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[j][m] = f32x4{0.f, 0.f, 0.f, 0.f};

  u32x4 wr[3][kWideNb];
  u32x4 xr[XP];
  load_x(xr, 0);
  load_w(wr[0], 0);
  load_w(wr[1], 1);
  store_x(xr, 0);
  load_x(xr, 1);
  sync();
  // sums of the runs so far: of the first TR row blocks in registers
  f32x4 tot_r[kWideNb][TR];
  auto tot = [&](int j, int m) -> f32x4& {
    return m < TR ? tot_r[j][m < TR ? m : 0] : tot_l[(j * (MT - TR) + m - TR) * 64];
  };
#pragma unroll
  for (int j = 0; j < kWideNb; ++j)
#pragma unroll
    for (int m = 0; m < MT; ++m) tot(j, m) = acc[j][m];
  auto step = [&](int i, const u32x4 (&wc)[kWideNb], u32x4 (&wnext)[kWideNb]) {
    load_w(wnext, i + 2);
    const u32x4* xb = xs + (i & 1) * XT * 64 + lane;
    u32x4 f[2][2];
    f[0][0] = xb[0];
    f[0][1] = xb[64];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m + 1 < MT) {
        f[(m + 1) & 1][0] = xb[(2 * m + 2) * 64];
        f[(m + 1) & 1][1] = xb[(2 * m + 3) * 64];
      }
      if (m == MT / 2) {
        store_x(xr, i + 1);
        load_x(xr, i + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kWideNb; ++j) acc[j][m] = mfma_bf16(as_bf16x8(wc[j]), as_bf16x8(f[m & 1][0]), acc[j][m]);
#pragma unroll
      for (int j = 0; j < kWideNb; ++j) acc[j][m] = mfma_bf16(as_bf16x8(wc[j]), as_bf16x8(f[m & 1][1]), acc[j][m]);
      __builtin_amdgcn_sched_barrier(0);
    }
    sync();
  };
  int trips = 0;
  for (int i = 0; i < n; i += 3) {
    step(i, wr[0], wr[2]);
    step(i + 1, wr[1], wr[0]);
    step(i + 2, wr[2], wr[1]);
    if (++trips == kWideRun / 3 && i + 3 < n) {
      trips = 0;
#pragma unroll
      for (int j = 0; j < kWideNb; ++j)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          tot(j, m) += acc[j][m];
          acc[j][m] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }

  // The K groups' partial tiles meet in LDS, two n-blocks of every wave a
  // round; then each wave sums whole tiles in group order and finishes them.
  f32x4* red = (f32x4*)sm;
  const EpiArgs& e = a.epi;
#pragma unroll
  for (int r = 0; r < kWideNb / 2; ++r) {
    if (r) __syncthreads();
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int m = 0; m < MT; ++m) red[((w * 2 + jj) * MT + m) * 64 + lane] = tot(2 * r + jj, m) + acc[2 * r + jj][m];
    __syncthreads();
    for (int it = w; it < 2 * NWN * MT; it += kWideWaves) {
      const int m = it % MT, wj = it / MT;             // wj = (wave along N) * 2 + jj
      const int nb = (nti * NWN + (wj >> 1)) * kWideNb + 2 * r + (wj & 1);
      const int mb = mb0 + m, mrow = mb * 16 + (lane & 15);
      if (nb >= a.Nb || mb >= Mb) continue;            // wave-uniform
      f32x4 v = red[(wj * MT + m) * 64 + lane];
#pragma unroll
      for (int g = 1; g < KG; ++g) v += red[((g * NWN * 2 + wj) * MT + m) * 64 + lane];
      if constexpr (EPI == EPI_TILE) {
        *(f32x4*)(e.out + split * e.part_stride + (((size_t)mb * a.Nb + nb) * 64 + lane) * 4) = v;
      } else if (mrow < a.M) {
        if constexpr (EPI == EPI_PART) {
          *(f32x4*)(e.out + split * e.part_stride + (size_t)mrow * e.ld + nb * 16 + (lane >> 4) * 4) = v;
        } else {
          EpiIn pre{};
          if constexpr (EPI == EPI_QKV) pre = qkv_inputs(e, nb, (lane >> 4) * 4, mrow);
          epilogue<W_BF16, EPI>(e, nb, (lane >> 4) * 4, mrow, split, v, pre);
        }
      }
    }
  }
}

// fp32 weights and activations: the window kernel's tile (16 features x 64
// rows, four waves splitting K as k_gemm_f32 does) over any number of row
// tiles, for models small enough that launches are most of what they cost.
template <int EPI>
__global__ __launch_bounds__(256) void k_gemm_wide_f32(GemmArgs a) {
  constexpr int NW = 4, MT = 4;
  __shared__ f32x4 red[NW * MT * 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nb = blockIdx.x, mb0 = blockIdx.y * MT, Mb = (a.M + 15) >> 4;
  const int per = (a.Kb + NW - 1) / NW, kb0 = min(a.Kb, w * per), kb1 = min(a.Kb, kb0 + per);
  const float4* __restrict__ W = (const float4*)a.W;
  const float4* __restrict__ X = (const float4*)a.Xhi;
  f32x4 acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = kb0; kb < kb1; ++kb) {
    const size_t wi = (((size_t)nb * a.Kb + kb) * 64 + lane) * 2;
    const F8 wf{W[wi], W[wi + 1]};
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const size_t xi = (((size_t)min(mb0 + t, Mb - 1) * a.Kb + kb) * 64 + lane) * 2;
      const F8 xf{X[xi], X[xi + 1]};
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};   // of this k-block
#pragma unroll
      for (int e = 0; e < 8; ++e) s = mfma_f32(f8_get(wf, e), f8_get(xf, e), s);
      acc[t] += s;
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) red[(w * MT + t) * 64 + lane] = acc[t];
  __syncthreads();
  // wave w finishes row tile w
  f32x4 v = red[w * 64 + lane];
#pragma unroll
  for (int i = 1; i < NW; ++i) v += red[(i * MT + w) * 64 + lane];
  const int m = (mb0 + w) * 16 + (lane & 15);
  if (m >= a.M) return;
  EpiIn pre{};
  if constexpr (EPI == EPI_QKV) pre = qkv_inputs(a.epi, nb, (lane >> 4) * 4, m);
  epilogue<W_F32, EPI>(a.epi, nb, (lane >> 4) * 4, m, 0, v, pre);
}

// sums the splits' tile-order partials (EPI_TILE) in split order and applies
// the role's epilogue; one wave per 16 x 16 tile
template <int EPI>
__global__ __launch_bounds__(256) void k_wide_fold(GemmArgs a, const float* part, size_t stride, int S) {
  const int lane = threadIdx.x & 63;
  const int nb = blockIdx.x * 4 + (threadIdx.x >> 6), mb = blockIdx.y;
  if (nb >= a.Nb) return;
  const float* p = part + (((size_t)mb * a.Nb + nb) * 64 + lane) * 4;
  f32x4 pv[kWideSplits];
#pragma unroll
  for (int s = 0; s < kWideSplits; ++s) pv[s] = *(const f32x4*)(p + min(s, S - 1) * stride);
  const int m = mb * 16 + (lane & 15);
  if (m >= a.M) return;
  EpiIn pre{};
  if constexpr (EPI == EPI_QKV) pre = qkv_inputs(a.epi, nb, (lane >> 4) * 4, m);
  f32x4 v = pv[0];
#pragma unroll
  for (int s = 1; s < kWideSplits; ++s)
    if (s < S) v += pv[s];
  epilogue<W_BF16, EPI>(a.epi, nb, (lane >> 4) * 4, m, 0, v, pre);
}

// ---------------------------------------------------------------- attention
//
// Causal attention of the prompt rows over the cache (the rows' own keys and
// values included: the QKV GEMM has written them).  Same arithmetic as the
// window kernel (attention.hip): S^T = K Q^T and O^T = V^T P^T in 16x16x32
// MFMAs, queries and probabilities split hi/lo, base-2 online softmax.
// Bound by the MFMAs, the fragment reads from LDS and the softmax arithmetic,
// about 1 us each per 64-key stage of a CU and only partly overlapped.  A unit is 16 consecutive rows of one head; a
// workgroup's 8 waves take 8 units that share keys (all heads of a KV group,
// row block by row block), so the keys and values of a 64-key stage are
// loaded once per workgroup into LDS, in fragment order, while the stage
// before is worked on, and a workgroup stops at its last row's position.
// 8B, 2048 rows: 97 us (5 % more with a maximum and a rescale per 32 keys),
// against 32 x 15 us of the window kernel, which reads the keys once per 16
// queries.
// With few row blocks the keys are cut into chunks as well (13B, 77 rows over
// 900 keys: 51 us whole, 19 + 5 in 256-key and 13 + 6 in 128-key chunks).
template <int KVB, int HD>
__global__ __launch_bounds__(512) void k_attn_prefill(AttnArgs a, int rb0, int n_units, int n_ublk) {
  constexpr int DS = HD / 32;
  constexpr int DT = HD / 16;
  constexpr int ST = 4 * DS;                 // tiles of a 32-key step: 2 DS of K, DT of V
  // a lane's eight elements of a tile: one 16-byte piece of a bf16 cache, two
  // of an fp32 cache
  struct Frag {
    u32x4 p[KVB ? 1 : 2];
  };
  __shared__ u32x4 kv[2][2 * ST][KVB ? 1 : 2][64];   // two stages of 64 keys
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kvh = blockIdx.x % a.n_kv, ic = blockIdx.x / a.n_kv;
  const int c = ic % a.n_chunks, ub = n_ublk - 1 - ic / a.n_chunks;   // longest first
  const int G = a.n_heads / a.n_kv, R = a.rows.rows_per_window;
  const int u = min(ub * 8 + w, n_units - 1), ul = min(ub * 8 + 7, n_units - 1);
  const bool live = ub * 8 + w < n_units;
  const int rb = rb0 + u / G, head = kvh * G + u % G;
  // position of the first row of a 16-row block (negative: rows of an invalid
  // group, whose output nobody reads), and the keys its rows see together:
  // [0, base + rows in it)
  auto block_pos = [&](int b) { return a.rows.gpos[b * 16 / kMaxRows] + b * 16 % kMaxRows; };
  auto block_keys = [&](int b) { return a.rows.gpos[b * 16 / kMaxRows] < 0 ? 0 : block_pos(b) + min(16, R - b * 16); };
  const int pos0 = block_pos(rb);
  const int kw = live ? block_keys(rb) : 0;             // keys of this wave
  int kwg = 0;                                          // and of the workgroup
  for (int b = rb0 + (ub * 8) / G; b <= rb0 + ul / G; ++b) kwg = max(kwg, block_keys(b));
  const int keys = a.rows.gpos[kGposKeys];
  const int per = a.n_chunks > 1 ? prefill_chunk(keys, a.n_chunks) >> 6 : 1 << 20;
  if (a.n_chunks > 1 && c * per * 64 >= keys && c > 0) return;   // no such chunk
  const int st0 = c * per, st1 = min((kwg + 63) >> 6, st0 + per);   // stages of 64 keys
  const int r16 = lane & 15, kgrp = (lane >> 4) * 8;
  const int row = rb * 16 + r16;
  const int qpos = pos0 + r16;
  const size_t base = ((size_t)a.rows.window0 * a.n_kv + kvh) * (size_t)a.maxlen * HD;
  constexpr int ESZ = KVB ? 2 : 4;
  const char* kc = (const char*)a.kc + base * ESZ;
  const char* vc = (const char*)a.vc + base * ESZ;
  const float scale2 = a.scale * 1.44269504088896340736f;   // log2 e

  // this wave's DS tiles of a stage: waves 0-3 the first 32 keys, 4-7 the
  // second; of each four, two load K (16-key halves), two V
  const int half = w >> 2, part = w & 3;
  auto load_stage = [&](Frag (&d)[DS], int st) {
    const int p0 = st * 64 + half * 32;
#pragma unroll
    for (int p = 0; p < DS; ++p) {
      const char* src = part < 2 ? kc + kc_off(p0 + (r16 >> 2) * 8 + part * 4 + (r16 & 3), p * 32 + kgrp, HD) * ESZ
                                 : vc + vc_off(p0 + kgrp, ((part - 2) * DS + p) * 16 + r16, HD) * ESZ;
      d[p] = *(const Frag*)src;
    }
  };
  auto store_stage = [&](const Frag (&d)[DS], int buf) {
#pragma unroll
    for (int p = 0; p < DS; ++p)
#pragma unroll
      for (int i = 0; i < (KVB ? 1 : 2); ++i) kv[buf][half * ST + part * DS + p][i][lane] = d[p].p[i];
  };

  const float* qrow = a.q + (size_t)min(row, R - 1) * (a.n_heads * HD) + head * HD;
  bf16x8 qh[DS], ql[DS];
  float qf[DS][8];
  Frag sr[DS];
  load_stage(sr, st0 < st1 ? st0 : 0);
#pragma unroll
  for (int ds = 0; ds < DS; ++ds) {
    const float4 a0 = *(const float4*)(qrow + ds * 32 + kgrp), a1 = *(const float4*)(qrow + ds * 32 + kgrp + 4);
    const float v[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    if constexpr (KVB) {
      u32x4 h, l;
      split8(v, h, l);
      qh[ds] = as_bf16x8(h);
      ql[ds] = as_bf16x8(l);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[ds][e] = v[e];
    }
  }
  float mrun = -INFINITY, lrun = 0.f;
  f32x4 o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto f32_at = [](const u32x4 (&x)[KVB ? 1 : 2][64], int lane, int e) {
    return __uint_as_float(x[KVB ? 0 : e >> 2][lane][e & 3]);
  };
  // one 64-key stage: both halves' scores, one maximum and one rescale, then
  // both halves' values.  Lane: keys p0 + 32 h + kgrp + e of query r16.
  auto stage = [&](int p0, const u32x4 (*tl)[KVB ? 1 : 2][64]) {
    f32x4 st[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        st[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
          if constexpr (KVB) {
            const bf16x8 kb = as_bf16x8(tl[h * ST + t * DS + ds][0][lane]);
            st[h][t] = mfma_bf16(kb, qh[ds], st[h][t]);
            st[h][t] = mfma_bf16(kb, ql[ds], st[h][t]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              st[h][t] = mfma_f32(f32_at(tl[h * ST + t * DS + ds], lane, e), qf[ds][e], st[h][t]);
          }
        }
      }
    const bool full = p0 + 64 <= pos0 + 1;
    // the maximum over the unscaled scores; the scale goes into the exponent
    float pv[2][8];
    float mloc = -INFINITY;
    if (full) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          pv[h][e] = st[h][e >> 2][e & 3];
          mloc = fmaxf(mloc, pv[h][e]);
        }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          pv[h][e] = p0 + 32 * h + kgrp + e <= qpos ? st[h][e >> 2][e & 3] : -INFINITY;
          mloc = fmaxf(mloc, pv[h][e]);
        }
    }
    const float mnew = fmaxf(mrun, max_over_16_32(mloc) * scale2);
    const float b = (mnew == -INFINITY) ? 0.f : mnew;
    float lsum = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pv[h][e] = __builtin_amdgcn_exp2f(fmaf(pv[h][e], scale2, -b));
        lsum += pv[h][e];
      }
    if (__ballot(mnew != mrun)) {
      const float alpha = __builtin_amdgcn_exp2f(mrun - b);
      lrun *= alpha;
#pragma unroll
      for (int t = 0; t < DT; ++t) o[t] *= alpha;
    }
    lrun += lsum;
    mrun = mnew;
    bf16x8 ph[2], pl[2];
    if constexpr (KVB) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u32x4 x, y;
        split8(pv[h], x, y);
        ph[h] = as_bf16x8(x);
        pl[h] = as_bf16x8(y);
      }
    }
    // keys past the block's rows may be dead cache rows: they have
    // probability 0, and their values are zeroed so that 0 * NaN never
    // reaches the output.  The values of a stage (of 32 keys of an fp32 cache)
    // are summed by themselves before they join the row's sum: one chain over
    // all keys left 9 % more error in the second layer's keys and values than
    // the window kernel (tiny fp32 model, 350 keys), this way 8 % less
    const int nv = kw - (p0 + kgrp);
    const bool tail = p0 + 64 > kw;
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if constexpr (KVB) {
          u32x4 vv = tl[h * ST + 2 * DS + t][0][lane];
          if (tail) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              vv[i] &= (2 * i < nv - 32 * h ? 0x0000FFFFu : 0u) | (2 * i + 1 < nv - 32 * h ? 0xFFFF0000u : 0u);
          }
          s = mfma_bf16(as_bf16x8(vv), ph[h], s);
          s = mfma_bf16(as_bf16x8(vv), pl[h], s);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float vv = f32_at(tl[h * ST + 2 * DS + t], lane, e);
            s = mfma_f32(e < nv - 32 * h ? vv : 0.f, pv[h][e], s);
          }
          if (h == 0) {
            o[t] += s;
            s = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        }
      }
      o[t] += s;
    }
  };

  store_stage(sr, 0);
  __syncthreads();
  for (int st = st0; st < st1; ++st) {
    const bool more = st + 1 < st1;
    if (more) load_stage(sr, st + 1);
    const int buf = (st - st0) & 1;
    if (st * 64 < kw) stage(st * 64, &kv[buf][0]);
    if (more) store_stage(sr, buf ^ 1);
    __syncthreads();
  }
  if (!live) return;
  lrun = sum_over_16_32(lrun);
  if (a.n_chunks > 1) {
    const size_t part = ((size_t)kvh * n_units + u) * a.n_chunks + c;
    float* po = a.part_o + (part * 16 + r16) * HD + (lane >> 4) * 4;
#pragma unroll
    for (int t = 0; t < DT; ++t) *(f32x4*)(po + t * 16) = o[t];
    if (lane < 16) a.part_ml[part * 16 + lane] = make_float2(mrun, lrun);   // base-2 units
    return;
  }
  if (row >= R) return;
  const float inv = 1.0f / lrun;
#pragma unroll
  for (int t = 0; t < DT; ++t) {
    const float y4[4] = {o[t][0] * inv, o[t][1] * inv, o[t][2] * inv, o[t][3] * inv};
    pack_store4(a.out, a.wtype, row, head * HD + t * 16 + (lane >> 4) * 4, y4);
  }
}

// sums the key chunks of one unit (16 rows of one head), chunks in order: one
// thread per row and four dims
template <int HD>
__global__ __launch_bounds__(HD * 4) void k_attn_prefill_combine(AttnArgs a, int rb0, int n_units) {
  const int kvh = blockIdx.x % a.n_kv, u = blockIdx.x / a.n_kv;
  const int G = a.n_heads / a.n_kv, R = a.rows.rows_per_window;
  const int q = threadIdx.x / (HD / 4), d = threadIdx.x % (HD / 4) * 4;
  const int row = (rb0 + u / G) * 16 + q;
  if (row >= R) return;
  const size_t part = ((size_t)kvh * n_units + u) * a.n_chunks;
  const float2* ml = a.part_ml + part * 16 + q;
  const float* po = a.part_o + (part * 16 + q) * HD + d;
  const int keys = a.rows.gpos[kGposKeys], per = prefill_chunk(keys, a.n_chunks);
  const int n_chunks = max(1, (keys + per - 1) / per);
  float M = -INFINITY;
  for (int c = 0; c < n_chunks; ++c) M = fmaxf(M, ml[c * 16].x);
  const float b = M == -INFINITY ? 0.f : M;
  float L = 0.f;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int c = 0; c < n_chunks; ++c) {
    const float2 v = ml[c * 16];
    const float f = __builtin_amdgcn_exp2f(v.x - b);
    L += v.y * f;
    acc += *(const f32x4*)(po + (size_t)c * 16 * HD) * f;
  }
  const float inv = 1.0f / L;
  const float y4[4] = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
  pack_store4(a.out, a.wtype, row, (kvh * G + u % G) * HD + d, y4);
}

}  // namespace

// NT variants of launches that no plan makes with one row tile are not built:
// eight waves along the features of O and down (at most 512 n-blocks, 16
// workgroups), four and eight of an unsplit QKV
template <int MT, int NWN, int NT>
hipError_t launch_wide_epi(const GemmArgs& a, const WideGrid& g, hipStream_t s) {
  const dim3 gd(g.per_xcd * 8), bd(kWideWaves * 64);
  constexpr int NT_PART = NWN == 8 ? 0 : NT, NT_QKV = NWN == 2 ? NT : 0;
  switch (a.epi.kind) {
    case EPI_PART: hipLaunchKernelGGL((k_gemm_wide<MT, NWN, EPI_PART, NT_PART>), gd, bd, 0, s, a, g); break;
    case EPI_TILE: hipLaunchKernelGGL((k_gemm_wide<MT, NWN, EPI_TILE, NT>), gd, bd, 0, s, a, g); break;
    case EPI_QKV: hipLaunchKernelGGL((k_gemm_wide<MT, NWN, EPI_QKV, NT_QKV>), gd, bd, 0, s, a, g); break;
    case EPI_SILU: hipLaunchKernelGGL((k_gemm_wide<MT, NWN, EPI_SILU, NT>), gd, bd, 0, s, a, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int MT>
hipError_t launch_wide_mt(const GemmArgs& a, int nwn, const WideGrid& g, hipStream_t s) {
  const bool one = g.mtiles == 1;
  if (nwn == 2) return one ? launch_wide_epi<MT, 2, 1>(a, g, s) : launch_wide_epi<MT, 2, 0>(a, g, s);
  if (nwn == 4) return one ? launch_wide_epi<MT, 4, 1>(a, g, s) : launch_wide_epi<MT, 4, 0>(a, g, s);
  return one ? launch_wide_epi<MT, 8, 1>(a, g, s) : launch_wide_epi<MT, 8, 0>(a, g, s);
}

hipError_t launch_gemm_wide(const GemmArgs& a, const WideCfg& c, hipStream_t s) {
  if (a.M < 1 || a.Nb < 1 || a.Kb < 1 || a.S < 1 || a.S > a.Kb || a.G < 1 || (c.nwn != 2 && c.nwn != 4 && c.nwn != 8))
    return hipErrorInvalidValue;
  if (a.S > 1 && a.epi.kind != EPI_PART && a.epi.kind != EPI_TILE) return hipErrorInvalidValue;
  WideGrid g;
  const int mb = (a.M + 15) / 16;
  g.mtiles = (mb + c.mt - 1) / c.mt;
  g.nt = (a.Nb + c.nwn * kWideNb - 1) / (c.nwn * kWideNb);
  g.tiles = g.nt * g.mtiles;
  g.per_xcd = (g.tiles * a.S + 7) / 8;
  switch (c.mt) {
    case 4: return launch_wide_mt<4>(a, c.nwn, g, s);
    case 5: return launch_wide_mt<5>(a, c.nwn, g, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_wide_f32(const GemmArgs& a, hipStream_t s) {
  if (a.M < 1 || a.Nb < 1 || a.Kb < 1 || a.S != 1 || a.G != 1) return hipErrorInvalidValue;
  const dim3 grid(a.Nb, (a.M + 63) / 64), blk(256);
  switch (a.epi.kind) {
    case EPI_PART: hipLaunchKernelGGL((k_gemm_wide_f32<EPI_PART>), grid, blk, 0, s, a); break;
    case EPI_QKV: hipLaunchKernelGGL((k_gemm_wide_f32<EPI_QKV>), grid, blk, 0, s, a); break;
    case EPI_SILU: hipLaunchKernelGGL((k_gemm_wide_f32<EPI_SILU>), grid, blk, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_wide_fold(const GemmArgs& a, const float* part, size_t stride, int S, hipStream_t s) {
  if (S < 1 || S > kWideSplits) return hipErrorInvalidValue;
  const dim3 grid((a.Nb + 3) / 4, (a.M + 15) / 16), blk(256);
  if (a.epi.kind == EPI_QKV) hipLaunchKernelGGL((k_wide_fold<EPI_QKV>), grid, blk, 0, s, a, part, stride, S);
  else if (a.epi.kind == EPI_SILU) hipLaunchKernelGGL((k_wide_fold<EPI_SILU>), grid, blk, 0, s, a, part, stride, S);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

int prefill_units(int rows, int group) { return (rows + 15) / 16 * group; }

template <int KVB, int HD>
hipError_t launch_attn_prefill_hd(const AttnArgs& a, int rb0, int units, hipStream_t s) {
  const int ub = (units + 7) / 8;
  hipLaunchKernelGGL((k_attn_prefill<KVB, HD>), dim3(ub * a.n_kv * a.n_chunks), dim3(512), 0, s, a, rb0, units, ub);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_chunks == 1) return e;
  hipLaunchKernelGGL((k_attn_prefill_combine<HD>), dim3(units * a.n_kv), dim3(HD * 4), 0, s, a, rb0, units);
  return hipGetLastError();
}

hipError_t launch_attention_prefill(int kv_bf16, int hd, const AttnArgs& a, int rb0, hipStream_t s) {
  const int units = prefill_units(a.rows.rows_per_window - 16 * rb0, a.n_heads / a.n_kv);
  if (rb0 < 0 || units < 1) return hipErrorInvalidValue;
  if (a.n_chunks < 1 || !a.rows.gpos) return hipErrorInvalidValue;
  if (kv_bf16) {
    switch (hd) {
      case 32: return launch_attn_prefill_hd<1, 32>(a, rb0, units, s);
      case 64: return launch_attn_prefill_hd<1, 64>(a, rb0, units, s);
      case 96: return launch_attn_prefill_hd<1, 96>(a, rb0, units, s);
      case 128: return launch_attn_prefill_hd<1, 128>(a, rb0, units, s);
    }
  } else {
    switch (hd) {
      case 32: return launch_attn_prefill_hd<0, 32>(a, rb0, units, s);
      case 64: return launch_attn_prefill_hd<0, 64>(a, rb0, units, s);
      case 96: return launch_attn_prefill_hd<0, 96>(a, rb0, units, s);
      case 128: return launch_attn_prefill_hd<0, 128>(a, rb0, units, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace dsi
