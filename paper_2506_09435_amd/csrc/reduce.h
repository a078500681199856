// reduce.h - block reductions of the vector kernels (device code), and the CG scalars taken from
// per-block partials.
//
// A kernel writes one FP64 partial per block and sum; the sums are formed in a fixed order, either by a
// one-block kernel or, where there are at most kFinPartials partials, by every block of the kernel
// that needs the result (all get the same bits).  The latter saves a launch, 4 us of the 27 us of a
// Jacobi CG iteration on the bar (64 x 16 x 4, p = 5); with the 6,554 partials of the sea's apply
// every block would read 52 KB, and the one-block kernel (8 us of 2 ms) is the cheaper one.
#pragma once

#include "fnpf_internal.h"

namespace fnpf {

constexpr int kFinPartials = 2048;

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block reduction of NS sums; thread 0 writes them to partial[blockIdx.x * NS + k].
template <int NS>
__device__ __forceinline__ void block_partials(double (&v)[NS], double *partial) {
  constexpr int NW = kVecThreads / 64;
  __shared__ double s[NS][NW];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    double r = wsum(v[k]);
    if (lane == 0) s[k][wv] = r;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      double a = 0.0;
      for (int w = 0; w < NW; ++w) a += s[k][w];
      partial[blockIdx.x * NS + k] = a;
    }
  }
}

// Fixed-order sum of per-thread values over the block; every thread gets it, and whether any wave's flag
// was set.
template <int NS>
__device__ __forceinline__ bool block_total(const double (&a)[NS], double (&out)[NS], bool flag = false) {
  constexpr int NW = kVecThreads / 64;
  __shared__ double s[NS][NW];
  __shared__ int any[NW];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) any[wv] = flag ? 1 : 0;
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const double r = wsum(a[k]);
    if (lane == 0) s[k][wv] = r;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    out[k] = 0.0;
    for (int w = 0; w < NW; ++w) out[k] += s[k][w];
  }
  int f = 0;
  for (int w = 0; w < NW; ++w) f |= any[w];
  return f != 0;
}

// Fixed-order sum of np partial tuples (stride NS) by one block; every thread gets it.
template <int NS>
__device__ __forceinline__ void final_sums(const double *partial, int np, double (&out)[NS]) {
  double a[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) a[k] = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < np; b += kVecThreads)
#pragma unroll
    for (int k = 0; k < NS; ++k) a[k] += partial[b * NS + k];
  block_total<NS>(a, out);
}

// The same for np <= kFinPartials in two steps, so that a kernel can issue these loads before its own
// and sum while the others are under way.
template <int NS>
struct PartialLoads {
  static constexpr int N = kFinPartials / kVecThreads;
  double v[N][NS];
  __device__ __forceinline__ PartialLoads(const double *partial, int np) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int b = threadIdx.x + m * kVecThreads;
#pragma unroll
      for (int k = 0; k < NS; ++k) v[m][k] = 0.0;
      if (m * kVecThreads < np && b < np) {
#pragma unroll
        for (int k = 0; k < NS; ++k) v[m][k] = partial[b * NS + k];
      }
    }
  }
  // true: one of the block's waves has seen the solve end (ended)
  __device__ __forceinline__ bool sums(double (&out)[NS], bool ended) const {
    double a[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      a[k] = v[0][k];   // (0 + v[0] would be formed, and the load waited for, ahead of the other loads)
#pragma unroll
      for (int m = 1; m < N; ++m) a[k] += v[m][k];
    }
    return block_total<NS>(a, out, ended);
  }
};

// alpha = r.z / p.Ap (0 on a breakdown, which ends the solve).  rz2 is the newest r.z; it becomes rz,
// which the direction update divides by.  Called by one thread.
__device__ __forceinline__ double cg_set_alpha(PcgScalars *sc, double pq, double rz) {
  double alpha = 0.0;
  sc->pq = pq;
  if (!(pq > 0.0) || !(pq <= 1e300)) {
    sc->breakdown = (pq == pq) ? 1 : 2;
    sc->done = 1;
  } else {
    alpha = rz / pq;
  }
  sc->alpha = alpha;
  sc->rz = rz;
  return alpha;
}

// The same by a whole grid: every block sums the partials of p.Ap, the first one stores.  False where
// nothing may be updated: on a breakdown, which leaves x at its last iterate, and where the solve has
// ended.  `ended` is the done flag as this wave read it: the first block may set it while the waves of
// another one start, some before and some after, so all of them go through the sum and leave together if
// one has seen it (a wave that left alone would leave its part of the sum unwritten).
__device__ __forceinline__ bool cg_alpha(const PartialLoads<1> &pq, bool ended, double rz, PcgScalars *sc,
                                         double &alpha) {
  double s[1];
  if (pq.sums(s, ended)) return false;
  if (blockIdx.x == 0 && threadIdx.x == 0) cg_set_alpha(sc, s[0], rz);
  alpha = rz / s[0];
  return s[0] > 0.0 && s[0] <= 1e300;
}

}  // namespace fnpf
