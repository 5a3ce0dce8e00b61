// Elementwise steps of the multigrid V-cycle (FP64 and FP32): D^-1 is one element's diagonal inverse (n3 values), the
// same on every element of a uniform periodic mesh; conversions between the
// FP64 outer CG and an FP32 cycle.
#include <hip/hip_runtime.h>

#include "cg_kernels.h"

namespace dgmf {

namespace {

constexpr int kThreads = kCgThreads;

// x = s D^-1 b
template <typename T>
__global__ void __launch_bounds__(kThreads) k_cheb_first(const T* __restrict__ b, const T* __restrict__ dinv, int n3,
                                                         T s, T* __restrict__ x, long long n) {
  for (long long i = blockIdx.x * (long long)kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads)
    x[i] = s * dinv[i % n3] * b[i];
}

// x += t
template <typename T>
__global__ void __launch_bounds__(kThreads) k_add(T* __restrict__ x, const T* __restrict__ t, long long n) {
  for (long long i = blockIdx.x * (long long)kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads)
    x[i] += t[i];
}

template <typename A, typename B>
__global__ void __launch_bounds__(kThreads) k_convert(const A* __restrict__ a, B* __restrict__ b, long long n) {
  for (long long i = blockIdx.x * (long long)kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads)
    b[i] = (B)a[i];
}

}  // namespace

hipError_t mg_cheb_first(const double* b, const double* dinv, int n3, double s, double* x, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_cheb_first<double>, dim3(kCgBlocks), dim3(kThreads), 0, st, b, dinv, n3, s, x, n);
  return hipGetLastError();
}
hipError_t mg_add(double* x, const double* t, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_add<double>, dim3(kCgBlocks), dim3(kThreads), 0, st, x, t, n);
  return hipGetLastError();
}

hipError_t mg_cheb_first(const float* b, const float* dinv, int n3, float s, float* x, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_cheb_first<float>, dim3(kCgBlocks), dim3(kThreads), 0, st, b, dinv, n3, s, x, n);
  return hipGetLastError();
}
hipError_t mg_add(float* x, const float* t, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_add<float>, dim3(kCgBlocks), dim3(kThreads), 0, st, x, t, n);
  return hipGetLastError();
}

hipError_t mg_convert(const double* a, float* b, long long n, hipStream_t st) {
  hipLaunchKernelGGL((k_convert<double, float>), dim3(kCgBlocks), dim3(kThreads), 0, st, a, b, n);
  return hipGetLastError();
}
hipError_t mg_convert(const float* a, double* b, long long n, hipStream_t st) {
  hipLaunchKernelGGL((k_convert<float, double>), dim3(kCgBlocks), dim3(kThreads), 0, st, a, b, n);
  return hipGetLastError();
}

}  // namespace dgmf
