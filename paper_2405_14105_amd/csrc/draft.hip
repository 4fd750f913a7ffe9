// Drafter sampling: from the drafter's logits of the row that ends the
// current context, the stored distribution q = softmax(z / T) (fp64, stored
// fp32) and the next draft, drawn from that stored row by inverse CDF
// (Section 2: the drafter proposes each lookahead token by sampling its own
// next-token distribution given the tokens before it).
//
// The draw: the smallest token t with sum_{v <= t} q_v > u * sum_v q_v, the
// sums taken in fp64 over the fp32 values in ascending token order; if
// rounding leaves no such t, the last t with q_t > 0.  Three launches, all
// with fixed reduction orders (run-to-run identical):
//   1. per 4096-entry chunk: max of z / T and sum of exp(z / T - max) (fp64);
//   2. per chunk: combine all chunk statistics (same order in every block),
//      write the chunk's q = (float) exp(z / T - M) / S, and the fp64 sum of
//      those fp32 values (per-thread runs of four, then a workgroup scan);
//   3. one workgroup: a wave prefix over the chunk sums locates the chunk
//      holding u * total, the chunk is rescanned in the same order, and the
//      token is written to its slot of the verification window.
#include <limits.h>
#include <math.h>

#include "scan.h"

namespace dsi {

namespace {

constexpr int ST = 1024;                 // threads per workgroup
constexpr int SW = ST / 64;              // waves
constexpr int SPER = kVerifyChunk / ST;  // consecutive entries per thread: four keep the chains short (see verify.hip)
static_assert(SPER == 4, "load_row4");

__global__ __launch_bounds__(ST) void k_dstat(DraftArgs a) {
  __shared__ double shd[SW];
  __shared__ float shv[SW];
  const int c = blockIdx.x;
  const int v0 = c * kVerifyChunk + threadIdx.x * SPER;
  float vals[SPER];
  load_row4(a.logits, v0, a.V, rows_aligned4(a.logits, a.V), vals);
  float zmax = -INFINITY;
#pragma unroll
  for (int i = 0; i < SPER; ++i) {
    if (v0 + i >= a.V) vals[i] = -INFINITY;
    zmax = fmaxf(zmax, vals[i]);
  }
  zmax = wave_max(zmax);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) shv[w] = zmax;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SW; ++i) zmax = fmaxf(zmax, shv[i]);
  const double m = over_t((double)zmax, a.temperature, a.inv_temperature);
  double sum = 0.0;
#pragma unroll
  for (int i = 0; i < SPER; ++i)
    if (v0 + i < a.V) sum += exp(over_t((double)vals[i], a.temperature, a.inv_temperature) - exp_base(m));
  sum = wave_sum(sum);
  if ((threadIdx.x & 63) == 0) shd[w] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    sum = shd[0];
#pragma unroll
    for (int i = 1; i < SW; ++i) sum += shd[i];
    a.part[c] = make_double2(m, sum);
  }
}

// the row's max and normaliser from the chunk statistics: wave 0, chunks
// lane, lane + 64, ... then a wave scan (every block computes the same)
__device__ __forceinline__ void row_stats(const DraftArgs& a, double* sM, double* sS) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    double m = -INFINITY;
    for (int c = lane; c < a.C; c += 64) m = fmax(m, a.part[c].x);
    m = wave_max(m);
    double s = 0.0;
    for (int c = lane; c < a.C; c += 64) s += a.part[c].y * exp(a.part[c].x - m);
    s = wave_sum(s);
    if (lane == 0) {
      *sM = m;
      *sS = s;
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(ST) void k_dq(DraftArgs a) {
  __shared__ double sM, sS;
  __shared__ double sh[SW];
  const int c = blockIdx.x;
  // thread t: entries c*4096 + 4 t .. +3 in order (the rescan's order)
  const int v0 = c * kVerifyChunk + threadIdx.x * SPER;
  float zv[SPER];
  load_row4(a.logits, v0, a.V, rows_aligned4(a.logits, a.V), zv);
  row_stats(a, &sM, &sS);
  const double M = sM, S = sS;
  double own = 0.0;
#pragma unroll
  for (int i = 0; i < SPER; ++i) {
    const int v = v0 + i;
    if (v < a.V) {
      const float q = (float)(exp(over_t((double)zv[i], a.temperature, a.inv_temperature) - M) / S);
      a.q_out[v] = q;
      own += (double)q;
    }
  }
  const double incl = block_scan_incl<SW>(own, sh);
  if (threadIdx.x == ST - 1) a.csum[c] = incl;
}

__global__ __launch_bounds__(ST) void k_ddraw(DraftArgs a) {
  __shared__ double sh[SW];
  __shared__ double sincl[ST];
  __shared__ double s_base, s_target;
  __shared__ int s_chunk;
  __shared__ int s_first[SW], s_last[SW];
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    // inclusive prefix over the chunk sums, 64 chunks at a time
    const double un = (double)a.u[0];
    auto prefix = [&](int g, double carry) {
      const int c = g * 64 + lane;
      double x = c < a.C ? a.csum[c] : 0.0;
      return carry + wave_scan_incl(x);
    };
    const int groups = (a.C + 63) / 64;
    const double incl0 = prefix(0, 0.0);
    double carry = lane_value(incl0, 63);
    for (int g = 1; g < groups; ++g) carry = lane_value(prefix(g, carry), 63);
    const double target = un * carry;
    int chunk = -1;
    double base = 0.0;
    carry = 0.0;
    for (int g = 0; g < groups; ++g) {
      const double incl = g == 0 ? incl0 : prefix(g, carry);
      const double prev = __shfl_up(incl, 1);
      const double excl = lane ? prev : carry;   // exact prefix before chunk g*64+lane
      const unsigned long long hit = __ballot(g * 64 + lane < a.C && incl > target);
      if (hit) {   // uniform across the wave
        const int l = __ffsll((long long)hit) - 1;
        chunk = g * 64 + l;
        base = lane_value(excl, l);
        break;
      }
      carry = lane_value(incl, 63);
    }
    if (chunk < 0) {
      // rounding left no crossing: the last chunk with mass (drawn from its
      // last nonzero entry below)
      for (int c = a.C - 1; c >= 0; --c)
        if (a.csum[c] > 0.0) {
          chunk = c;
          break;
        }
      if (chunk < 0) chunk = a.C - 1;
      base = INFINITY;   // no entry crosses
    }
    if (lane == 0) {
      s_chunk = chunk;
      s_base = base;
      s_target = target;
    }
  } else if (threadIdx.x < 128 && a.lens) {
    // wave 1: the forwarded rows (at most 64) enter the drafter's cache if
    // every id is valid; the first step's last one is w0
    const int lane = threadIdx.x - 64;
    const int t = lane < a.n_rows ? a.rows[lane] : 0;
    const bool bad = __any(t < 0 || t >= a.V);
    if (lane == 0) {
      if (bad) atomicOr(a.err, 1);
      else a.lens[a.window] += a.n_rows;
    }
    if (a.w0_out && lane == a.n_rows - 1) *a.w0_out = t;
  }
  __syncthreads();
  const int v0 = s_chunk * kVerifyChunk + threadIdx.x * SPER;
  double vals[SPER];
  double own = 0.0;
  int lastpos = -1;
  // all loads first (clamped index, masked after): a wait behind a
  // conditional load is a wait for every load issued before it
  float qv[SPER];
  load_row4(a.q_out, v0, a.V, rows_aligned4(a.q_out, a.V), qv);
#pragma unroll
  for (int i = 0; i < SPER; ++i) {
    const int v = v0 + i;
    vals[i] = v < a.V ? (double)qv[i] : 0.0;
    own += vals[i];
    if (vals[i] > 0.0) lastpos = v;
  }
  const double incl = block_scan_incl<SW>(own, sh);
  sincl[threadIdx.x] = incl;
  __syncthreads();
  int first = INT_MAX;
  if (s_base != INFINITY) {
    double cw = threadIdx.x > 0 ? sincl[threadIdx.x - 1] : 0.0;
#pragma unroll
    for (int i = 0; i < SPER; ++i) {
      cw += vals[i];
      if (first == INT_MAX && s_base + cw > s_target && vals[i] > 0.0) first = v0 + i;
    }
  }
  int tok = block_first_or_last<SW>(first, lastpos, s_first, s_last);
  if (threadIdx.x == 0) {
    if (tok < 0) tok = 0;
    *a.tok_out = tok;
  }
}

}  // namespace

size_t draft_workspace_bytes(int V) {
  const int C = (V + kVerifyChunk - 1) / kVerifyChunk;
  return (size_t)C * (sizeof(double2) + sizeof(double)) + 256;
}

hipError_t launch_draft_sample(DraftArgs a, void* ws, hipStream_t s) {
  if (a.lens && (a.n_rows < 1 || a.n_rows > kMaxRows)) return hipErrorInvalidValue;
  a.C = (a.V + kVerifyChunk - 1) / kVerifyChunk;
  a.inv_temperature = 1.0 / a.temperature;
  a.part = (double2*)ws;
  a.csum = (double*)((char*)ws + (((size_t)a.C * sizeof(double2) + 15) & ~(size_t)15));
  hipLaunchKernelGGL(k_dstat, dim3(a.C), dim3(ST), 0, s, a);
  hipLaunchKernelGGL(k_dq, dim3(a.C), dim3(ST), 0, s, a);
  hipLaunchKernelGGL(k_ddraw, dim3(1), dim3(ST), 0, s, a);
  return hipGetLastError();
}

}  // namespace dsi
