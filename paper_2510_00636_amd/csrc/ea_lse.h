// Log-sum-exps of a head from its (max, sum exp) partials, in index order whatever made them.
#pragma once
#include <hip/hip_runtime.h>

namespace ea {

template <typename LT>
struct LT2;
template <>
struct LT2<float> { typedef float2 type; };
template <>
struct LT2<double> { typedef double2 type; };

__device__ __forceinline__ float ea_exp(float x) { return expf(x); }
__device__ __forceinline__ double ea_exp(double x) { return exp(x); }
__device__ __forceinline__ float ea_log(float x) { return logf(x); }
__device__ __forceinline__ double ea_log(double x) { return log(x); }

template <typename LT>
__device__ __forceinline__ void merge_lt(LT& m, LT& s, LT m2, LT s2) {
  LT mn = m > m2 ? m : m2;
  if (mn == -INFINITY) { s = 0; m = mn; }
  else { s = s * ea_exp(m - mn) + s2 * ea_exp(m2 - mn); m = mn; }
}

// (max, sum exp) of partials c0, c0 + step, .. of a head: four at a time, requested together, the largest maximum first
// and one exponential per partial then (merged one by one they cost two exponentials and a memory latency each).
template <typename LT>
__device__ __forceinline__ void gather_lt(const typename LT2<LT>::type* __restrict__ p, int npart, int c0, int step, LT& m, LT& s) {
  constexpr int U = 4;
  m = -INFINITY;
  s = 0;
  if (npart <= step) {                      // one, or none
    if (c0 < npart) { m = p[c0].x; s = p[c0].y; }
    return;
  }
  for (int c = c0; c < npart; c += U * step) {
    typename LT2<LT>::type x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x[u] = p[min(c + u * step, npart - 1)];
      if (c + u * step >= npart) x[u].x = -INFINITY;
    }
    LT mn = m;
#pragma unroll
    for (int u = 0; u < U; ++u) mn = mn > x[u].x ? mn : x[u].x;
    if (mn == -INFINITY) continue;
    s *= ea_exp(m - mn);
#pragma unroll
    for (int u = 0; u < U; ++u) s += c + u * step < npart ? x[u].y * ea_exp(x[u].x - mn) : (LT)0;
    m = mn;
  }
}

// log-sum-exp of one head from its npart partials, by one wavefront: lane l takes partials
// l, l + 64, ... in increasing order, then a fixed butterfly over the lanes.
template <typename LT>
__device__ __forceinline__ LT wave_lse(const typename LT2<LT>::type* __restrict__ p, int npart, int lane) {
  LT m, s;
  gather_lt<LT>(p, npart, lane, 64, m, s);
  for (int o = 32; o >= 1; o >>= 1) {
    LT m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o);
    merge_lt<LT>(m, s, m2, s2);
  }
  return m + ea_log(s);
}

}  // namespace ea
