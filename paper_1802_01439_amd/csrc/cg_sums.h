// Final sums of a reduction's partials by one workgroup (device code of the
// CG scalar kernels).
#pragma once

#include <hip/hip_runtime.h>

namespace dgmf {

// One workgroup on an idle device: bound by the latency of its loads, so 16
// wavefronts with four loads in flight each (256 threads in a plain loop took
// 25.9 us for the 2 x 10368 partials of a dual-splitting velocity solve at
// k = 7, 24^3, this takes SUMS_US).
constexpr int kSumThreads = 1024;

// Sums of partial[q * nblocks + i] over i for q < NQ, in a fixed order
// (thread-strided, then across the wavefront, then across the wavefronts);
// valid in thread 0.
template <int NQ>
__device__ __forceinline__ void block_sums(const double* __restrict__ partial, int nblocks, double (&out)[NQ]) {
  constexpr int W = kSumThreads / 64, U = 4;
  __shared__ double sh[NQ][W];
  double s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = 0.0;
  for (int i0 = threadIdx.x; i0 < nblocks; i0 += U * kSumThreads) {
    double v[U][NQ];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * kSumThreads, nblocks - 1);
#pragma unroll
      for (int q = 0; q < NQ; ++q) v[u][q] = partial[(size_t)q * nblocks + i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) s[q] += i0 + u * kSumThreads < nblocks ? v[u][q] : 0.0;
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
    out[q] = sh[q][0];
#pragma unroll
    for (int w = 1; w < W; ++w) out[q] += sh[q][w];
  }
}

}  // namespace dgmf
