// Accept/reject of B verification windows from their target logits.
//
// Sampling mode (the lossless rule the paper adopts from its cited works,
// Sections 2 and 3.1), per window with rows z_0..z_k:
//   p_i = softmax(z_{i-1} / T); a_i = p_i(d_i) / q_i(d_i); A_i = [u_i < a_i];
//   n = min{i : A_i = 0} - 1 (else k), the accepted count of Theorem 2's
//   proof; token drawn by inverse CDF with u_{k+1} from max(0, p_{n+1} -
//   q_{n+1}) (n < k; p_{n+1} if that has no mass) or from p_{k+1} (n = k).
// Greedy mode (Algorithm 1's exact match): A_i = [d_i = argmax z_{i-1}],
//   token = argmax z_n, ties to the lowest id.
// All softmax statistics, ratios and CDF sums are fp64 (an fp32 CDF over
// 128k entries picks visibly different tokens); every reduction has a fixed
// order, so results are run-to-run identical.
//
// Four launches:
//   1. row statistics: per (row, 4096-entry chunk) max, sum exp, argmax;
//   2. decide: one workgroup per window, a wave per row combines the chunk
//      statistics, then one wave tests the k drafts in parallel and finds the
//      first rejection with a ballot; greedy windows finish here;
//   3. per (window, chunk): fp64 sums of the residual (and of p) over the
//      chunk, via the same block scan used in step 4;
//   4. sample: one workgroup per window locates the chunk that holds
//      u_{k+1} R, rescans it and emits the token; commits the KV length.
#include <limits.h>
#include <math.h>

#include "scan.h"

namespace dsi {

namespace {

constexpr int VT = 1024;                 // threads per workgroup
constexpr int VW = VT / 64;              // waves
constexpr int PER = kVerifyChunk / VT;   // consecutive entries per thread
static_assert(PER == 4, "load_row4");

// A chunk is 4096 entries, four per thread: the kernels are chains of loads,
// fp64 exponentials and reductions, and four entries a thread instead of 16
// shorten every link (7 windows x 6 rows x 128256 entries: 49 -> 33 us for the
// four launches).  The row statistics of many (row, chunk) pairs are bound
// by how many loads the waves in flight hold instead; there a thread takes the
// entries of 1024 / THR threads, each summed as if it had a thread of its own,
// so that a row's statistics are the same bits either way.
template <int THR>
__global__ __launch_bounds__(THR) void k_vrow(VerifyArgs a) {
  constexpr int NV = VT / THR;
  __shared__ double shd[VW];
  __shared__ float shv[THR / 64];
  __shared__ int shi[THR / 64];
  const int c = blockIdx.x, r = blockIdx.y;
  const float* z = a.logits + (size_t)r * a.V;
  const bool vec = rows_aligned4(a.logits, a.V);
  const int v0 = c * kVerifyChunk + threadIdx.x * PER;
  float vals[NV][PER];
#pragma unroll
  for (int g = 0; g < NV; ++g) load_row4(z, v0 + g * THR * PER, a.V, vec, vals[g]);
  float zmax = -INFINITY;
  int zarg = INT_MAX;
#pragma unroll
  for (int g = 0; g < NV; ++g)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int v = v0 + g * THR * PER + i;
      if (v < a.V) take_max(zmax, zarg, vals[g][i], v);
    }
  wave_argmax(zmax, zarg);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    shv[w] = zmax;
    shi[w] = zarg;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < THR / 64; ++i) take_max(zmax, zarg, shv[i], shi[i]);
  double m = 0.0;
  if (!a.greedy) {   // the exact-match rules read the argmax only
    m = over_t((double)zmax, a.temperature, a.inv_temperature);
    const double mb = exp_base(m);
#pragma unroll
    for (int g = 0; g < NV; ++g) {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (v0 + g * THR * PER + i < a.V)
          sum += exp(over_t((double)vals[g][i], a.temperature, a.inv_temperature) - mb);
      sum = wave_scan_incl(sum);
      if (lane == 63) shd[g * (THR / 64) + w] = sum;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (!a.greedy) {
      double sum = shd[0];
#pragma unroll
      for (int i = 1; i < VW; ++i) sum += shd[i];
      a.part[(size_t)r * a.C + c] = make_double2(m, sum);
    }
    a.part_arg[(size_t)r * a.C + c] = make_float2(zmax, __int_as_float(zarg));
  }
}

// one workgroup per window: each wave combines the chunk statistics of a
// row (lanes over chunks, a wave scan in fixed order), then wave 0 decides; its
// drafts' q and logits are requested before the statistics
__global__ __launch_bounds__(VT) void k_vdecide(VerifyArgs a) {
  __shared__ double sM[kMaxRows], sS[kMaxRows];
  __shared__ int sArg[kMaxRows];
  const int b = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = a.k, R = k + 1;
  int bad = 0, d = 0;
  float qd = 1.f, zd = 0.f, ud = 0.f;
  if (w == 0) {
    if (lane < R) {
      const int t = a.tokens[b * R + lane];
      if (t < 0 || t >= a.V) bad = 1;
    }
    if (lane < k) {
      d = a.tokens[b * R + lane + 1];
      const int dc = d < 0 || d >= a.V ? 0 : d;   // an id outside the vocabulary is reported by its own row
      if (!a.greedy) {
        qd = a.q[((size_t)b * k + lane) * a.V + dc];
        zd = a.logits[(size_t)(b * R + lane) * a.V + dc];
        ud = a.u[b * R + lane];
      }
    }
  }
  for (int i = w; i < R; i += VW) {
    const int r = b * R + i;
    double m = -INFINITY, sum = 0.0;
    float bv = -INFINITY;
    int bi = INT_MAX;
    for (int c = lane; c < a.C; c += 64) {
      const float2 pa = a.part_arg[(size_t)r * a.C + c];
      if (!a.greedy) m = fmax(m, a.part[(size_t)r * a.C + c].x);
      take_max(bv, bi, pa.x, __float_as_int(pa.y));
    }
    if (!a.greedy) {
      m = wave_max(m);
      for (int c = lane; c < a.C; c += 64) {
        const double2 pc = a.part[(size_t)r * a.C + c];
        sum += pc.y * exp(pc.x - m);
      }
      sum = wave_sum(sum);
    }
    wave_argmax(bv, bi);
    if (lane == 0) {
      sM[i] = m;
      sS[i] = sum;
      sArg[i] = bi;
      a.rowstat[r] = make_double2(m, sum);
      a.rowarg[r] = bi;
    }
  }
  __syncthreads();
  if (w != 0) return;
  const int arg = lane < R ? sArg[lane] : 0;
  bool acc = true;
  if (lane < k && !bad) {
    if (a.greedy) {
      acc = (d == arg);
    } else if (!(qd > 0.f) || !isfinite(qd)) {
      bad = 1;
    } else {
      const double p = exp(over_t((double)zd, a.temperature, a.inv_temperature) - sM[lane]) / sS[lane];
      acc = (double)ud < p / (double)qd;
    }
  }
  const bool anybad = __any(bad);
  const unsigned long long rej = __ballot(lane < k && !acc);
  const int n = rej ? (__ffsll((long long)rej) - 1) : k;
  const int tokn = __shfl(arg, n);
  if (lane == 0) {
    if (anybad) {
      a.n_out[b] = -1;
      a.tok_out[b] = -1;
      atomicOr(a.err, 2);
      a.decision[b] = make_int4(n, b * R + n, 0, 1);
    } else if (a.greedy) {
      a.n_out[b] = n;
      a.tok_out[b] = tokn;
      if (a.commit && a.lens) a.lens[a.window0 + b] += n + 1;
      a.decision[b] = make_int4(n, b * R + n, 0, 1);
    } else {
      a.decision[b] = make_int4(n, b * R + n, n < k ? 1 : 0, 0);
    }
  }
}

// p_v of an entry with logit z, and its mass in the window's drawing
// distribution
__device__ __forceinline__ double entry_p(const VerifyArgs& a, float z, double M, double S) {
  return exp(over_t((double)z, a.temperature, a.inv_temperature) - M) / S;
}
__device__ __forceinline__ double entry_mass(double p, float q, bool residual) {
  if (!residual) return p;
  const double d = p - (double)q;
  return d > 0.0 ? d : 0.0;
}

// the PER logits and, when qrow is given, drafter probabilities from entry v0 on
__device__ __forceinline__ void load_entries(const VerifyArgs& a, const float* zrow, const float* qrow, int v0,
                                             float (&zv)[PER], float (&qv)[PER]) {
  load_row4(zrow, v0, a.V, rows_aligned4(a.logits, a.V), zv);
  if (qrow) {
    load_row4(qrow, v0, a.V, rows_aligned4(a.q, a.V), qv);
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) qv[i] = 0.f;
  }
}

__global__ __launch_bounds__(VT) void k_vresid(VerifyArgs a) {
  __shared__ double sh[2 * VW];
  const int c = blockIdx.x, b = blockIdx.y;
  const int4 dec = a.decision[b];
  if (dec.w) return;
  const int n = dec.x, r = dec.y;
  const bool residual = dec.z != 0;
  const double2 st = a.rowstat[r];
  const float* zrow = a.logits + (size_t)r * a.V;
  const float* qrow = residual ? a.q + ((size_t)b * a.k + n) * a.V : nullptr;
  const int v0 = c * kVerifyChunk + threadIdx.x * PER;
  float zv[PER], qv[PER];
  load_entries(a, zrow, qrow, v0, zv, qv);
  double sr = 0.0, sp = 0.0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (v0 + i < a.V) {
      const double p = entry_p(a, zv[i], st.x, st.y);
      sr += entry_mass(p, qv[i], residual);
      sp += p;
    }
  }
  block_scan_incl2<VW>(sr, sp, sh);
  if (threadIdx.x == VT - 1) a.csum[(size_t)b * a.C + c] = make_double2(sr, sp);
}

__global__ __launch_bounds__(VT) void k_vsample(VerifyArgs a) {
  __shared__ double sh[VW];
  __shared__ double s_base, s_target;
  __shared__ int s_chunk, s_usep, s_found;
  __shared__ int s_first[VW], s_last[VW];
  const int b = blockIdx.x;
  const int4 dec = a.decision[b];
  if (dec.w) return;
  const int n = dec.x, r = dec.y;
  const bool residual0 = dec.z != 0;
  const double2 st = a.rowstat[r];
  if (threadIdx.x < 64) {
    // wave 0: prefix sums over the chunk sums, 64 chunks at a time, in one
    // fixed order for the total and for locating the chunk
    const int lane = threadIdx.x;
    const int groups = (a.C + 63) / 64;
    const double un = a.u[b * (a.k + 1) + a.k];
    double2 cs0 = make_double2(0.0, 0.0);   // the first 64 chunks: all of them up to 262144 entries
    if (lane < a.C) cs0 = a.csum[(size_t)b * a.C + lane];
    auto prefix = [&](int g, double carry, int usep) {
      const int c = g * 64 + lane;
      double x = 0.0;
      if (g == 0) {
        x = usep ? cs0.y : cs0.x;
      } else if (c < a.C) {
        const double2 cs = a.csum[(size_t)b * a.C + c];
        x = usep ? cs.y : cs.x;
      }
      return carry + wave_scan_incl(x);
    };
    int usep = 0;
    double incl0 = prefix(0, 0.0, 0);
    double R = lane_value(incl0, 63);
    for (int g = 1; g < groups; ++g) R = lane_value(prefix(g, R, 0), 63);
    if (residual0 && !(R > 0.0)) {   // no residual mass: draw from p
      usep = 1;
      incl0 = prefix(0, 0.0, 1);
      R = lane_value(incl0, 63);
      for (int g = 1; g < groups; ++g) R = lane_value(prefix(g, R, 1), 63);
    }
    const double target = un * R;
    int chunk = -1;
    double base = 0.0, carry = 0.0;
    for (int g = 0; g < groups; ++g) {
      const double incl = g == 0 ? incl0 : prefix(g, carry, usep);
      const double prev = __shfl_up(incl, 1);
      const double excl = lane ? prev : carry;
      const unsigned long long hit = __ballot(g * 64 + lane < a.C && incl > target);
      if (hit) {   // uniform across the wave
        const int l = __ffsll((long long)hit) - 1;
        chunk = g * 64 + l;
        base = lane_value(excl, l);
        break;
      }
      carry = lane_value(incl, 63);
    }
    int found = 1;
    if (chunk < 0) {               // rounding left no crossing: last chunk with mass
      found = 0;
      for (int c = a.C - 1; c >= 0; --c) {
        const double2 cs = a.csum[(size_t)b * a.C + c];
        if ((usep ? cs.y : cs.x) > 0.0) {
          chunk = c;
          break;
        }
      }
      if (chunk < 0) chunk = a.C - 1;
    }
    if (lane == 0) {
      s_chunk = chunk;
      s_base = base;
      s_target = target;
      s_usep = usep;
      s_found = found;
    }
  }
  __syncthreads();
  const bool residual = residual0 && !s_usep;
  const float* zrow = a.logits + (size_t)r * a.V;
  const float* qrow = residual ? a.q + ((size_t)b * a.k + n) * a.V : nullptr;
  const int v0 = s_chunk * kVerifyChunk + threadIdx.x * PER;
  float zv[PER], qv[PER];
  load_entries(a, zrow, qrow, v0, zv, qv);
  double vals[PER];
  double own = 0.0;
  int lastpos = -1;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int v = v0 + i;
    vals[i] = v < a.V ? entry_mass(entry_p(a, zv[i], st.x, st.y), qv[i], residual) : 0.0;
    own += vals[i];
    if (vals[i] > 0.0) lastpos = v;
  }
  const double incl = block_scan_incl<VW>(own, sh);
  // exclusive prefix of this thread = inclusive prefix of the previous one
  __shared__ double sincl[VT];
  sincl[threadIdx.x] = incl;
  __syncthreads();
  double run = s_base + (threadIdx.x > 0 ? sincl[threadIdx.x - 1] : 0.0);
  int first = INT_MAX;
  if (s_found) {
    double cw = threadIdx.x > 0 ? sincl[threadIdx.x - 1] : 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      cw += vals[i];
      run = s_base + cw;
      if (first == INT_MAX && run > s_target && vals[i] > 0.0) first = v0 + i;
    }
  }
  int tok = block_first_or_last<VW>(first, lastpos, s_first, s_last);
  if (threadIdx.x == 0) {
    if (tok < 0) tok = 0;
    a.n_out[b] = n;
    a.tok_out[b] = tok;
    if (a.commit && a.lens) a.lens[a.window0 + b] += n + 1;
  }
}

}  // namespace

size_t verify_workspace_bytes(int rows, int B, int V) {
  const int C = (V + kVerifyChunk - 1) / kVerifyChunk;
  size_t s = 0;
  s += (size_t)rows * C * sizeof(double2);   // part
  s += (size_t)rows * C * sizeof(float2);    // part_arg
  s += (size_t)rows * sizeof(double2);       // rowstat
  s += (size_t)rows * sizeof(int) + 16;      // rowarg
  s += (size_t)B * sizeof(int4);             // decision
  s += (size_t)B * C * sizeof(double2);      // csum
  return s + 256;
}

void verify_bind_workspace(VerifyArgs& a, void* ws, int rows, int B, int V) {
  a.inv_temperature = 1.0 / a.temperature;
  const int C = (V + kVerifyChunk - 1) / kVerifyChunk;
  char* p = (char*)ws;
  auto take = [&](size_t bytes) {
    char* q = p;
    p += (bytes + 15) & ~(size_t)15;
    return q;
  };
  a.C = C;
  a.part = (double2*)take((size_t)rows * C * sizeof(double2));
  a.part_arg = (float2*)take((size_t)rows * C * sizeof(float2));
  a.rowstat = (double2*)take((size_t)rows * sizeof(double2));
  a.rowarg = (int*)take((size_t)rows * sizeof(int));
  a.decision = (int4*)take((size_t)B * sizeof(int4));
  a.csum = (double2*)take((size_t)B * C * sizeof(double2));
}

// Up to 512 (row, chunk) pairs fit the CUs as 1024-thread workgroups; more of
// them run faster with 16 entries a thread (42 rows of 128256 entries, 1344
// pairs: 15.9 against 22.1 us).
hipError_t launch_verify_rowstats(const VerifyArgs& a, hipStream_t s) {
  const int rows = a.B * (a.k + 1);
  const dim3 grid(a.C, rows);
  if ((long long)a.C * rows <= 512) hipLaunchKernelGGL((k_vrow<VT>), grid, dim3(VT), 0, s, a);
  else hipLaunchKernelGGL((k_vrow<256>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_verify(const VerifyArgs& a, hipStream_t s) {
  const hipError_t e = launch_verify_rowstats(a, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_vdecide, dim3(a.B), dim3(VT), 0, s, a);
  if (!a.greedy) {
    hipLaunchKernelGGL(k_vresid, dim3(a.C, a.B), dim3(VT), 0, s, a);
    hipLaunchKernelGGL(k_vsample, dim3(a.B), dim3(VT), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace dsi
