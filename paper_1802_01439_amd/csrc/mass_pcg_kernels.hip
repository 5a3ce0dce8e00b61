// Scalar steps of the inverse-mass-preconditioned CG with its scalars kept on
// the device (the state array of the CG solver: kRZ, kBeta, kRN2, kDone,
// kStatus, kIter, kTol2, kMaxIt), so that iterations run in batches between
// host reads.  p.Ap and alpha come from the CG kernels, the r update with
// z = M^-1 r and the sums r.r, r.z from the fused inverse mass kernel.
#include "cg_kernels.h"
#include "cg_sums.h"

namespace dgmf {

namespace {

constexpr int kThreads = kCgThreads;

// r.z of the initial residual
__global__ void __launch_bounds__(kSumThreads) k_mp_start(const double* __restrict__ partial, int nblocks,
                                                          double* __restrict__ st) {
  double v[1];
  block_sums<kSumThreads, 1>(partial, nblocks, v);
  const double rz = v[0];
  if (threadIdx.x != 0) return;
  st[kRZ] = rz;
  if (!(rz > 0.0) || !isfinite(rz)) {
    st[kDone] = 1.0;
    st[kStatus] = 2.0;
  }
}

// after the r update and z = M^-1 r, with their partials r.r and r.z:
// convergence test, iteration count, beta
template <int TH>
__global__ void __launch_bounds__(TH) k_mp_beta(const double* __restrict__ partial, int nblocks,
                                                double* __restrict__ st) {
  double v[2];
  block_sums<TH, 2>(partial, nblocks, v);
  const double rr = v[0], rz = v[1];
  if (threadIdx.x != 0) return;
  if (st[kDone] != 0.0) {
    st[kBeta] = 0.0;
    return;
  }
  const double it = st[kIter] + 1.0;
  st[kIter] = it;
  st[kRN2] = rr;
  st[kBeta] = 0.0;
  if (rr <= st[kTol2]) {
    st[kDone] = 1.0;
    return;
  }
  if (it >= st[kMaxIt]) {
    st[kDone] = 1.0;
    st[kStatus] = 1.0;
    return;
  }
  if (!(rz > 0.0) || !isfinite(rz)) {
    st[kDone] = 1.0;
    st[kStatus] = 2.0;
    return;
  }
  st[kBeta] = rz / st[kRZ];
  st[kRZ] = rz;
}

// x += alpha p, then p = z + beta p (scalars from the state).  x moves here and
// not with r, because p is read here anyway: 4 + 5 vectors per iteration in
// the two kernels instead of 7 + 3.
template <int R>
__global__ void __launch_bounds__(kThreads) k_mp_update_xp(double* __restrict__ x, double* __restrict__ p,
                                                           const double* __restrict__ z,
                                                           const double* __restrict__ st, long long n) {
  step_xp<R>(x, p, z, st[kAlpha], st[kBeta], 0.0, n);
}

}  // namespace

hipError_t mpcg_start(const double* partial, double* st, hipStream_t s) {
  hipLaunchKernelGGL(k_mp_start, dim3(1), dim3(kSumThreads), 0, s, partial, kCgBlocks, st);
  return hipGetLastError();
}

hipError_t mpcg_beta(const double* partial, int nblocks, double* st, hipStream_t s) {
  if (nblocks > kManySums)
    hipLaunchKernelGGL(k_mp_beta<kManySumThreads>, dim3(1), dim3(kManySumThreads), 0, s, partial, nblocks, st);
  else
    hipLaunchKernelGGL(k_mp_beta<kSumThreads>, dim3(1), dim3(kSumThreads), 0, s, partial, nblocks, st);
  return hipGetLastError();
}

hipError_t mpcg_update_xp(double* x, double* p, const double* z, const double* st, long long n, hipStream_t s) {
  hipLaunchKernelGGL(xp_in_cache(n) ? k_mp_update_xp<2> : k_mp_update_xp<1>, dim3(kCgBlocks), dim3(kThreads), 0, s, x,
                     p, z, st, n);
  return hipGetLastError();
}

}  // namespace dgmf
