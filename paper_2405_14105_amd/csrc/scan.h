// Wave and workgroup reductions and scans of the accept/reject and drafter
// sampling kernels, which are chains of them: DPP steps take a few cycles each
// where a shuffle goes through LDS.
#pragma once

#include <limits.h>
#include <math.h>

#include "device_util.h"

namespace dsi {

// A lane's value from another lane by DPP (no LDS round trip); lanes that the
// pattern gives no source, or whose row is not in ROWS, get `old`.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_from(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_from(float old, float x) {
  return __int_as_float(dpp_from<CTRL, ROWS>(__float_as_int(old), __float_as_int(x)));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from(double old, double x) {
  return __hiloint2double(dpp_from<CTRL, ROWS>(__double2hiint(old), __double2hiint(x)),
                          dpp_from<CTRL, ROWS>(__double2loint(old), __double2loint(x)));
}
// Calls f(control, rows) for the six steps after which lane l has met lanes
// 0..l: shifts by 1, 2, 4, 8 within rows of 16 lanes, then lane 15 of a row
// to the row after it, then lane 31 to the upper half.
template <int N>
struct DppStep {
  static constexpr int ctrl = N == 0 ? 0x111 : N == 1 ? 0x112 : N == 2 ? 0x114 : N == 3 ? 0x118 : N == 4 ? 0x142 : 0x143;
  static constexpr int rows = N == 4 ? 0xA : N == 5 ? 0xC : 0xF;
};
template <int N = 0, typename F>
__device__ __forceinline__ void dpp_steps(F&& f) {
  f(DppStep<N>{});
  if constexpr (N < 5) dpp_steps<N + 1>(f);
}
__device__ __forceinline__ double wave_scan_incl(double v) {
  dpp_steps([&](auto s) { v += dpp_from<decltype(s)::ctrl, decltype(s)::rows>(0.0, v); });
  return v;
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ double wave_sum(double v) { return lane_value(wave_scan_incl(v), 63); }
__device__ __forceinline__ double wave_max(double v) {
  dpp_steps([&](auto s) { v = fmax(v, dpp_from<decltype(s)::ctrl, decltype(s)::rows>(v, v)); });
  return lane_value(v, 63);
}
__device__ __forceinline__ float wave_max(float v) {
  dpp_steps([&](auto s) { v = fmaxf(v, dpp_from<decltype(s)::ctrl, decltype(s)::rows>(v, v)); });
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// the larger value, ties to the smaller index
__device__ __forceinline__ void take_max(float& v, int& i, float ov, int oi) {
  if (ov > v || (ov == v && oi < i)) {
    v = ov;
    i = oi;
  }
}
__device__ __forceinline__ void wave_argmax(float& v, int& i) {
  dpp_steps([&](auto s) {
    const float ov = dpp_from<decltype(s)::ctrl, decltype(s)::rows>(v, v);
    const int oi = dpp_from<decltype(s)::ctrl, decltype(s)::rows>(i, i);
    take_max(v, i, ov, oi);
  });
  v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
  i = __builtin_amdgcn_readlane(i, 63);
}

// inclusive scan of one double per thread over a workgroup of NW waves, with a
// fixed association (wave scan, then the wave totals in order); sh holds NW
// doubles.  Every thread of the workgroup must call it.
template <int NW>
__device__ __forceinline__ double waves_before(const double* sh, int w) {
  double off = 0.0;
#pragma unroll
  for (int i = 0; i < NW - 1; ++i) {
    const double x = sh[i];
    off += i < w ? x : 0.0;
  }
  return off;
}
template <int NW>
__device__ __forceinline__ double block_scan_incl(double v, double* sh) {
  const int w = threadIdx.x >> 6;
  v = wave_scan_incl(v);
  if ((threadIdx.x & 63) == 63) sh[w] = v;
  __syncthreads();
  const double off = waves_before<NW>(sh, w);
  __syncthreads();
  return off + v;
}
// two scans at once (the same association each); sh holds 2 NW doubles
template <int NW>
__device__ __forceinline__ void block_scan_incl2(double& a, double& b, double* sh) {
  const int w = threadIdx.x >> 6;
  a = wave_scan_incl(a);
  b = wave_scan_incl(b);
  if ((threadIdx.x & 63) == 63) {
    sh[w] = a;
    sh[NW + w] = b;
  }
  __syncthreads();
  a += waves_before<NW>(sh, w);
  b += waves_before<NW>(sh + NW, w);
  __syncthreads();
}

// The first `first` (else the last `last`) of the workgroup's threads in thread
// order; threads without one pass INT_MAX (-1).  sf, sl hold NW ints; the
// result is thread 0's.  Ballots and one slot per wave: an LDS atomic a thread
// on one word runs its 1024 lanes one after another.
template <int NW>
__device__ __forceinline__ int block_first_or_last(int first, int last, int* sf, int* sl) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long f = __ballot(first != INT_MAX), l = __ballot(last >= 0);
  if (f == 0) {
    if (lane == 0) sf[w] = INT_MAX;
  } else if (lane == __ffsll((long long)f) - 1) {
    sf[w] = first;
  }
  if (l == 0) {
    if (lane == 0) sl[w] = -1;
  } else if (lane == 63 - __clzll((long long)l)) {
    sl[w] = last;
  }
  __syncthreads();
  int a = INT_MAX, b = -1;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    a = min(a, sf[i]);
    b = max(b, sl[i]);
  }
  return a != INT_MAX ? a : b;
}

// z / T with inv = 1 / T: the product corrected by its remainder (Markstein's
// division step), for a fraction of the division's instructions; exact at T
// = 1, and infinities and NaN as the division gives them
__device__ __forceinline__ double over_t(double z, double t, double inv) {
  const double q = z * inv;
  return __builtin_isfinite(q) ? fma(fma(-q, t, z), inv, q) : q;
}

// What is subtracted from a chunk's exponents, the largest of which is m: in a
// chunk of masked entries (all -inf) not -inf itself, so that each adds exp(-inf)
// = 0 and not exp(-inf + inf)
__device__ __forceinline__ double exp_base(double m) { return m == -INFINITY ? 0.0 : m; }

// Entries v .. v + 3 of a row of n values, all in flight together: one
// 16-byte load where `vec` says that rows are 16-byte aligned and n a multiple
// of four, else single loads with the index clamped into the row (entries past
// it are never used)
__device__ __forceinline__ void load_row4(const float* row, int v, int n, bool vec, float (&x)[4]) {
  if (vec) {
    const float4 f = *(const float4*)(row + min(v, n - 4));
    x[0] = f.x;
    x[1] = f.y;
    x[2] = f.z;
    x[3] = f.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = row[min(v + i, n - 1)];
  }
}
__device__ __forceinline__ bool rows_aligned4(const float* p, int n) {
  return (n & 3) == 0 && ((uintptr_t)p & 15) == 0;
}

}  // namespace dsi
