// Multigrid smoother work fused into the epilogue of the Laplace apply
// (Sec. 3.3, the V-cycle's Chebyshev smoother from a zero start), FP64 and
// FP32.  A step needs no vector of its own for the step direction, since
// that is the difference of the last two iterates:
//   x_{j+1} = x_j + c1 (x_j - x_{j-1}) + c2 D^-1 (b - A x_j),
// and the first iterate x_1 = s D^-1 b is formed from b wherever it is read:
//   first   x_2 from b alone              (reads b, writes x_2)
//   second  x_3, x_1 formed from b        (reads x_2, b, writes x_3)
//   later   x_{j+1} over x_{j-1}          (reads x_j, x_{j-1}, b, writes)
//   added   the last step of the post-smoothing, y += x_{j+1}
//   residual  res = b - A x
// The operand x_j is read for neighbour DoFs by other workgroups, x_{j-1} only
// by the thread that owns each DoF, which overwrites it.  D^-1 is one
// element's diagonal inverse, indexed by the local node.
// Bound: HBM.  A smoothing of degree 5 moves 13 vectors (23 with the step
// direction stored, x_1 written by a kernel of its own), the post-smoothing
// with its residual 17 (26 before).  The first step's two loads per neighbour
// value cost registers (FP64 n = 9 195 against 140, two wavefronts per SIMD
// instead of three; FP32 n = 9 108 / 72) and about a fifth of its own time, but
// a whole cycle is faster at every degree, us: FP64 k = 1, 64^3 534 -> 444,
// k = 4, 32^3 865 -> 665, k = 8, 16^3 824 -> 718, k = 11, 12^3 844 -> 767; FP32
// 402 -> 374, 639 -> 557, 591 -> 522, 593 -> 520.
// Rounding: the step x_j - x_{j-1} of two rounded iterates carries the rounding
// of x, a stored direction that of its own size.  In FP32 cycles against FP64
// ones the two forms are equally far off, also over many steps (medians of 16
// inputs, k = 3: degrees 5 / 10 1.9e-7 both, 30 / 100 4.6e-7 stored, 4.4e-7
// here; k = 7 1.3e-7, 3.8e-7 and 3.7e-7).
#include "laplace_kernels.h"
#include "ops.h"

namespace dgmf {

namespace {

enum { kFirst, kSecond, kLater };

template <typename T, int KIND, bool ADD>
struct MgChebIO {
  const T* x;   // operand (unused by the first step)
  const T* b;
  const T* __restrict__ dinv;
  const T* prev;   // x_{j-1} (later steps); out may be the same vector
  T* out;
  T s, c1, c2;
  __device__ __forceinline__ void begin() {}
  __device__ __forceinline__ T load(size_t i, int loc) const {
    if constexpr (KIND == kFirst) return s * dinv[loc] * b[i];
    else return x[i];
  }
  __device__ __forceinline__ void store(size_t i, int loc, T in, T ax) {
    const T bi = b[i], di = dinv[loc];
    T step = in;   // x_j - x_{j-1}
    if constexpr (KIND == kSecond) step -= s * di * bi;
    if constexpr (KIND == kLater) step -= prev[i];
    const T xn = in + (c1 * step + c2 * di * (bi - ax));
    if constexpr (ADD) out[i] += xn;
    else out[i] = xn;
  }
  template <int THREADS, size_t BYTES>
  __device__ __forceinline__ void finish(void*) {}
};

template <typename T>
struct MgResIO {
  const T* __restrict__ x;
  const T* __restrict__ b;
  T* __restrict__ res;
  __device__ __forceinline__ void begin() {}
  __device__ __forceinline__ T load(size_t i, int) const { return x[i]; }
  __device__ __forceinline__ void store(size_t i, int, T, T out) { res[i] = b[i] - out; }
  template <int THREADS, size_t BYTES>
  __device__ __forceinline__ void finish(void*) {}
};

template <typename T, typename IO>
hipError_t dispatch(const LaplacePlan& P, const IO& io, hipStream_t s) {
  switch (P.k) {
    case 1: return launch_laplace_io<2, T>(P, io, nullptr, s);
    case 2: return launch_laplace_io<3, T>(P, io, nullptr, s);
    case 3: return launch_laplace_io<4, T>(P, io, nullptr, s);
    case 4: return launch_laplace_io<5, T>(P, io, nullptr, s);
    case 5: return launch_laplace_io<6, T>(P, io, nullptr, s);
    case 6: return launch_laplace_io<7, T>(P, io, nullptr, s);
    case 7: return launch_laplace_io<8, T>(P, io, nullptr, s);
    case 8: return launch_laplace_io<9, T>(P, io, nullptr, s);
    case 9: return launch_laplace_io<10, T>(P, io, nullptr, s);
    case 10: return launch_laplace_io<11, T>(P, io, nullptr, s);
    case 11: return launch_laplace_io<12, T>(P, io, nullptr, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <typename T>
hipError_t mg_apply_cheb(const LaplacePlan& P, const MgChebStep<T>& st, hipStream_t s) {
  if (!st.x) {
    if (st.add) return hipErrorInvalidValue;
    return dispatch<T>(P, MgChebIO<T, kFirst, false>{nullptr, st.b, st.dinv, nullptr, st.out, st.s, st.c1, st.c2}, s);
  }
  if (!st.prev) {
    if (st.add) return hipErrorInvalidValue;
    return dispatch<T>(P, MgChebIO<T, kSecond, false>{st.x, st.b, st.dinv, nullptr, st.out, st.s, st.c1, st.c2}, s);
  }
  if (st.add)
    return dispatch<T>(P, MgChebIO<T, kLater, true>{st.x, st.b, st.dinv, st.prev, st.out, st.s, st.c1, st.c2}, s);
  return dispatch<T>(P, MgChebIO<T, kLater, false>{st.x, st.b, st.dinv, st.prev, st.out, st.s, st.c1, st.c2}, s);
}

template <typename T>
hipError_t mg_apply_residual(const LaplacePlan& P, const T* x, const T* b, T* res, hipStream_t s) {
  MgResIO<T> io{x, b, res};
  return dispatch<T>(P, io, s);
}

template hipError_t mg_apply_cheb<double>(const LaplacePlan&, const MgChebStep<double>&, hipStream_t);
template hipError_t mg_apply_cheb<float>(const LaplacePlan&, const MgChebStep<float>&, hipStream_t);
template hipError_t mg_apply_residual<double>(const LaplacePlan&, const double*, const double*, double*, hipStream_t);
template hipError_t mg_apply_residual<float>(const LaplacePlan&, const float*, const float*, float*, hipStream_t);

}  // namespace dgmf
