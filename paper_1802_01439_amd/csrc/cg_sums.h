// Code shared by the CG kernels: the update of solution and direction, and the
// final sums of a reduction's partials by one workgroup.
#pragma once

#include <hip/hip_runtime.h>

#include "cg_kernels.h"

namespace dgmf {

// x += alpha p, then p = (z - mu) + beta p: a zero alpha touches no x, a zero
// beta never uses the old direction for p.  A thread loads R entries of the
// grid-stride loop before it uses them: R = 2 while x, p and z stay in the
// last-level cache (256 MB) between kernels, where the loop is bound by its
// loads' latency (FP64 z, 2.7M entries 19.2 -> 16.5 us; FP32 z, 7.1M entries
// 50.0 -> 39.1); from memory R = 1 is faster (21M entries 101 against 115 us).
inline bool xp_in_cache(long long n) { return 24 * n <= 256LL << 20; }

template <int R, typename T>
__device__ __forceinline__ void step_xp(double* __restrict__ x, double* __restrict__ p, const T* __restrict__ z,
                                        double alpha, double beta, double mu, long long n) {
  const long long S = (long long)gridDim.x * kCgThreads;
  long long i = blockIdx.x * (long long)kCgThreads + threadIdx.x;
  if constexpr (R > 1) {
    for (; i + (R - 1) * S < n; i += R * S) {
      double zi[R], pi[R], xi[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        zi[u] = (double)z[i + u * S] - mu;
        pi[u] = p[i + u * S];
      }
      if (alpha != 0.0) {
#pragma unroll
        for (int u = 0; u < R; ++u) xi[u] = x[i + u * S];
#pragma unroll
        for (int u = 0; u < R; ++u) x[i + u * S] = xi[u] + alpha * pi[u];
      }
#pragma unroll
      for (int u = 0; u < R; ++u) p[i + u * S] = beta != 0.0 ? zi[u] + beta * pi[u] : zi[u];
    }
  }
  for (; i < n; i += S) {
    const double zi = (double)z[i] - mu;
    if (alpha != 0.0 || beta != 0.0) {
      const double pi = p[i];
      if (alpha != 0.0) x[i] += alpha * pi;
      p[i] = beta != 0.0 ? zi + beta * pi : zi;
    } else {
      p[i] = zi;
    }
  }
}

// Threads of a final sum.  One workgroup on an idle device, bound by the
// latency of its loads: four in flight per thread and quantity (two for three
// and more quantities in 1024 threads, for the registers), and 16 wavefronts only
// for many partials, since they cost more to start and to combine.  256 against
// 1024 threads, us: four quantities of 1024 partials 2.7 / 5.0, three 2.3 / 4.1,
// two 2.1 / 3.3; one of 4096 2.8 / 2.3, three 3.5 / 4.6; two of 10368 (a
// dual-splitting velocity solve, k = 7, 24^3) 5.8 / 5.2, of 30000 13.7 / 10.4
// (256 threads in a plain loop: 1024 partials 2.1-3.2, 10368 12.7).
constexpr int kSumThreads = 256, kManySumThreads = 1024, kManySums = 4096;

// Sums of partial[q * nblocks + i] over i for q < NQ, in a fixed order
// (thread-strided, then across the wavefront, then across the wavefronts);
// valid in thread 0.
template <int TH, int NQ>
__device__ __forceinline__ void block_sums(const double* __restrict__ partial, int nblocks, double (&out)[NQ]) {
  constexpr int W = TH / 64, U = TH == kManySumThreads && NQ > 2 ? 2 : 4;
  __shared__ double sh[NQ][W];
  double s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = 0.0;
  for (int i0 = threadIdx.x; i0 < nblocks; i0 += U * TH) {
    double v[U][NQ];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * TH, nblocks - 1);
#pragma unroll
      for (int q = 0; q < NQ; ++q) v[u][q] = partial[(size_t)q * nblocks + i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) s[q] += i0 + u * TH < nblocks ? v[u][q] : 0.0;
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
  }
  if (threadIdx.x % 64 == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) sh[q][threadIdx.x / 64] = s[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    out[q] = sh[q][threadIdx.x % W];
#pragma unroll
    for (int o = W / 2; o > 0; o >>= 1) out[q] += __shfl_xor(out[q], o, 64);
  }
}

}  // namespace dgmf
