// Operator of the projection step (Sec. 3.3: (M + A_D + A_C) u; the penalty
// terms of Sec. 3.2): mass, divergence penalty (div v, tau_D div u)_K and
// continuity penalty (v . n, {tau_C} [[u]] . n) on the faces, for a velocity
// field, FP64 and FP32, degrees 1..11, k+1 Gauss points per direction.
//
// Work in the Lagrange basis of the Gauss points (the k+1 point rule makes
// the interpolation S: LGL -> Gauss square and the quadrature exact):
//   ug_j = (S (x) S (x) S) u_j,
//   div  = sum_j (1/h_j) Dg_j ug_j         (Dg: collocation derivative),
//   z_j  = vol W ug_j + (1/h_j) Dg_j^T (tau_D vol W div),
//   y_j  = (S^T (x) S^T (x) S^T) z_j  + continuity term,
// where W is the tensor Gauss weight.  On a face normal to e_d only the
// normal component couples: y_d gains area {tau_C} (M1 (x) M1)(u^-_d - u^+_d)
// on the face layer (LGL face nodes, M1 the 1D mass on [0,1]).
//
// Component j is swept along its two tangential directions first and along
// e_j last.  The same two sweeps over the jumps u^-_j - u^+_j of the nodes on
// the two faces normal to e_j give the jumps at the tangential Gauss points.
// With M1 = S^T W S the term area {tau_C} W (u^-_j - u^+_j) is added after the
// S^T sweep along e_j, and the two tangential S^T sweeps finish it: no face
// mass products.  Along e_j, S and Dg (and Dg^T and S^T) run on one pencil in
// registers.  The jumps are formed at the nodes, from the loaded values: as
// the difference of two swept traces a small jump would carry the rounding of
// the traces, which strong penalties multiply.
//
// Mapping: one workgroup per batch of E elements, n^2 threads per component
// (one per pencil); batches are mapped XCD-aware, so that the neighbours'
// facing layers are mostly found in the same L2.  The first sweep runs on
// pencils loaded from memory, the last on pencils stored to it, the others on
// LDS pencils in place; 6 barriers.  Both point sets are symmetric about 1/2,
// so S and S^T are centrosymmetric and Dg, Dg^T centro-antisymmetric: every 1D
// sweep runs in even-odd form, about half the multiply-adds of the dense
// product.
//
// What bounds it: vector instructions (FP64 48-66 % of the time at four cycles
// each, FP32 77-100 %) and LDS (23-40 % resp. 34-64 %, its conflicts with it)
// together; memory sees each value read and written once.
// Measured with three sets of vectors in turn, FP64, against sweeps in the
// order x, y, z for all components with the face terms from two products with
// M1: k = 3, 32^3 45.9 -> 38.4 us, k = 6, 19x18x17 44.5 -> 34.3, k = 7, 24^3
// 124 -> 94, k = 9, 16^3 113 -> 71, k = 11, 12^3 68 -> 54; FP32 k = 7, 24^3
// 66 -> 56.  Jumps of swept traces instead of swept jumps would take 2-5 % less
// at k = 6, where they are loaded apart, and the same or more elsewhere.  (For
// k = 6, 10, 11: taking the own layers from LDS in the next phase instead of
// loading them again was 0-6 % slower.)
#include <algorithm>
#include <cmath>

#include "api_internal.h"
#include "common.h"
#include "laplace_kernels.h"
#include "ops.h"

namespace dgmf {

namespace {

// Even-odd form of an n x n matrix A with A[n-1-i][n-1-j] = SIG A[i][j]
// (H = n/2): P[i][j] = (A[i][j] + A[i][n-1-j]) / 2, Q[i][j] = (A[i][j] -
// A[i][n-1-j]) / 2 for i, j < H; for odd n also the middle column, row and
// entry.
template <int N, typename T>
struct EOMat {
  static constexpr int H = N / 2;
  T P[H][H], Q[H][H];
  T col[H], row[H], mid;
};

// y = A x for such a matrix, from the even and odd halves of x.
template <int N, int SIG, typename T, typename M>
__device__ __forceinline__ void eo_apply(const M& A, const T* x, T* y) {
  constexpr int H = N / 2;
  T e[H], o[H];
#pragma unroll
  for (int j = 0; j < H; ++j) {
    e[j] = x[j] + x[N - 1 - j];
    o[j] = x[j] - x[N - 1 - j];
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    T P = A.P[i][0] * e[0];
#pragma unroll
    for (int j = 1; j < H; ++j) P = fmadd(A.P[i][j], e[j], P);
    if constexpr (N % 2) P = fmadd(A.col[i], x[H], P);
    T Q = A.Q[i][0] * o[0];
#pragma unroll
    for (int j = 1; j < H; ++j) Q = fmadd(A.Q[i][j], o[j], Q);
    y[i] = P + Q;
    y[N - 1 - i] = SIG > 0 ? P - Q : Q - P;
  }
  if constexpr (N % 2) {
    T m = A.mid * x[H];
#pragma unroll
    for (int j = 0; j < H; ++j) m = fmadd(A.row[j], SIG > 0 ? e[j] : o[j], m);
    y[H] = m;
  }
}

template <int N, typename T>
struct ProjTab {
  EOMat<N, T> S, St, Dg, Dt;   // S[q][a] = l_a(z_q); Dg[q][r] = derivative of
                               // the Gauss Lagrange basis r at z_q; St, Dt transposed
  T w[N];                      // Gauss weights on [0,1]
  T vol, ih[3], area[3];
};

// LDS layout of one element.  Every component j keeps its block by role: t2
// innermost, then t1, then the direction n normal to its faces (e_j), with the
// jumps to the neighbours' facing layers at both ends (n + 2 layers).  t1 is the first
// tangential direction swept (z; y for j = 2), t2 the second (x; y for j = 0).
// So the sweeps run at strides known at compile time, and an odd stride of t1
// keeps them nearly free of bank conflicts.  Then the six face factors.
template <int N>
struct ProjCfg {
  static constexpr int N2 = N * N, N3 = N * N * N, M = N + 2;
  // The first two sweeps cover n + 2 layers: n^2 threads per component take
  // their own layers, and those with a pencil on a face its jump too (of the
  // values they have loaded); or n (n + 2) threads take one pencil each.  The
  // second way costs another wavefront at most n (n = 8: 4 instead of 3), which
  // measured slower up to n = 10 (n = 6 120 against 104 us at 32^3, n = 8 102 /
  // 95 at 24^3, n = 9 55 / 45 at 16^3), but none at n = 7 (34.9 / 35.3), and for
  // n = 11, 12 it is one in eight (54 / 60, 54 / 56).
  static constexpr bool TWO = N <= 10 && N != 7;
  static constexpr int TC = TWO ? N2 : N * M;
  // elements per workgroup: full wavefronts, and no more of them than needed
  // to hide the barriers (twice these were 10-30 % slower at n = 2..6)
  static constexpr int E = N == 2 ? 16 : N == 3 ? 7 : N == 4 ? 4 : N == 5 ? 3 : 1;
  static constexpr int THREADS = E * 3 * TC;
  static constexpr int S1 = N | 1, SN = N * S1;
  static constexpr int CP = M * SN;                 // one component
  static constexpr int FC = 3 * CP, PER = FC + 6;
};

template <int N, typename T>
__global__ void __launch_bounds__(ProjCfg<N>::THREADS)
projection_kernel(const T* __restrict__ u, T* __restrict__ y, const T* __restrict__ tau_d,
                  const T* __restrict__ tau_c, MeshArgs mesh, const ProjTab<N, T>* __restrict__ tab,
                  T* __restrict__ dot) {
  using C = ProjCfg<N>;
  constexpr int N2 = C::N2, N3 = C::N3, M = C::M, TC = C::TC, E = C::E;
  constexpr int S1 = C::S1, SN = C::SN;
  __shared__ T lds[E * C::PER];
  const int tid = threadIdx.x;
  const size_t cs = (size_t)mesh.n_el * N3;
  const int e0 = xcd_remap(blockIdx.x, gridDim.x) * E;
  auto pick = [](int j, int a0, int a1, int a2) { return j == 0 ? a0 : j == 1 ? a1 : a2; };
  // ---- P0, P1: S along t1 and t2 of the n + 2 layers
  {
    const int le = E == 1 ? 0 : tid / (3 * TC), rem = tid - le * 3 * TC;
    const int j = rem / TC, p = rem - j * TC;
    const int e = e0 + le;
    const bool active = e < mesh.n_el;
    T* A = lds + le * C::PER + j * C::CP;
    // pencil t of layer lay of element el, along t1
    auto load = [&](int el, int lay, int t, T (&x)[N]) {
      const T* g = u + j * cs + (size_t)el * N3 + pick(j, lay + N * t, t + N * lay, t + N2 * lay);
      const int gs = j == 2 ? N : N2;
#pragma unroll
      for (int c = 0; c < N; ++c) x[c] = g[gs * c];
    };
    // S along t1 of a pencil into position t of layer q
    auto sweep1 = [&](int q, int t, const T (&x)[N]) {
      T v[N];
      eo_apply<N, 1>(fresh(tab)->S, x, v);
      T* a = A + SN * q + t;
#pragma unroll
      for (int c = 0; c < N; ++c) a[S1 * c] = v[c];
    };
    auto sweep2 = [&](int q, int t) {
      T* a = A + SN * q + S1 * t;
      T x[N], v[N];
#pragma unroll
      for (int c = 0; c < N; ++c) x[c] = a[c];
      eo_apply<N, 1>(fresh(tab)->S, x, v);
#pragma unroll
      for (int c = 0; c < N; ++c) a[c] = v[c];
    };
    if (active) {
      // the neighbours across the two faces normal to e_j (periodic)
      const unsigned nxy = mesh.nx * mesh.ny;
      const unsigned ez = (unsigned)e / nxy, exy = (unsigned)e - ez * nxy;
      const unsigned ey = exy / (unsigned)mesh.nx, ex = exy - ey * mesh.nx;
      const int ej = pick(j, ex, ey, ez), last = pick(j, mesh.nx, mesh.ny, mesh.nz) - 1;
      const int step = pick(j, 1, mesh.nx, nxy);
      const int nl = e + (ej == 0 ? last : -1) * step, nr = e + (ej == last ? -last : 1) * step;
      auto factor = [&](int s) {
        lds[le * C::PER + C::FC + 2 * j + s] = T(0.5) * (tau_c[e] + tau_c[s ? nr : nl]) * tab->area[j];
      };
      if constexpr (C::TWO) {
        const int a = p % N, b = p / N;   // lanes run along x first
        const int lay = j == 0 ? a : b, t = j == 0 ? b : a;
        const bool edge = lay == 0 || lay == N - 1;
        T x[N], h[N];
        load(e, lay, t, x);
        if (edge) {
          load(lay ? nr : nl, N - 1 - lay, t, h);
          if (t == 0) factor(lay != 0);
#pragma unroll
          for (int c = 0; c < N; ++c) h[c] = x[c] - h[c];
        }
        sweep1(1 + lay, t, x);
        if (edge) sweep1(lay ? M - 1 : 0, t, h);
      } else {
        const int q = j == 0 ? p % M : p / N, t = j == 0 ? p / M : p % N;
        const bool jump = q == 0 || q == M - 1;
        const int lay = q == 0 ? 0 : q == M - 1 ? N - 1 : q - 1;
        T x[N], h[N];
        load(e, lay, t, x);
        if (jump) {
          load(q ? nr : nl, N - 1 - lay, t, h);
          if (t == 0) factor(q != 0);
#pragma unroll
          for (int c = 0; c < N; ++c) x[c] -= h[c];
        }
        sweep1(q, t, x);
      }
    }
    __syncthreads();
    if (active) {
      if constexpr (C::TWO) {
        sweep2(1 + p / N, p % N);
        if (p < 2 * N) sweep2(p < N ? 0 : M - 1, p % N);
      } else {
        sweep2(p / N, p % N);
      }
    }
    __syncthreads();
  }
  // ---- from here n^2 threads per component
  const int le = E == 1 ? 0 : tid / (3 * N2), rem = tid - le * 3 * N2;
  const int j = rem / N2, p = rem - j * N2;
  const int p0 = p % N, p1 = p / N;
  const int e = e0 + le;
  const bool active = tid < E * 3 * N2 && e < mesh.n_el;
  T* L = lds + le * C::PER;
  T* A = L + j * C::CP;
  T* aj = A + p0 + S1 * p1;   // (t2, t1) = (p0, p1), from the jumps of the left face on
  // ---- P2: S along e_j; keep vol W ug_j in registers; the derivative
  //      (1/h_j) Dg_j ug_j goes back
  T mw[N];
  if (active) {
    const auto& t = *fresh(tab);
    T x[N], v[N];
#pragma unroll
    for (int r = 0; r < N; ++r) x[r] = aj[SN * (r + 1)];
    const T w2 = t.w[p0] * t.w[p1];   // tensor weight of the two fixed indices
    eo_apply<N, 1>(t.S, x, v);
    const T wv = t.vol * w2;
#pragma unroll
    for (int r = 0; r < N; ++r) mw[r] = wv * t.w[r] * v[r];
    eo_apply<N, -1>(t.Dg, v, x);
#pragma unroll
    for (int r = 0; r < N; ++r) aj[SN * (r + 1)] = t.ih[j] * x[r];
  }
  __syncthreads();
  // ---- P3: tau_D vol W div on this pencil (the sum over the components read by
  //      each of them: a block of its own in LDS for it was 0-10 % slower), then
  //      z_j = vol W ug_j + (1/h_j) Dg_j^T of it, S^T along e_j and the face
  //      terms on the two end nodes
  if (active) {
    const auto& t = *fresh(tab);
    T x[N], v[N];
    // this pencil in the block of component k with strides sx, sy, sz
    auto block = [&](int k, int sx, int sy, int sz) {
      return L + k * C::CP + SN + pick(j, sy * p0 + sz * p1, sx * p0 + sz * p1, sx * p0 + sy * p1);
    };
    const T *a0 = block(0, SN, 1, S1), *a1 = block(1, 1, SN, S1), *a2 = block(2, 1, S1, SN);
    const int s0 = pick(j, SN, 1, S1), s1 = pick(j, 1, SN, S1), s2 = pick(j, 1, S1, SN);
    const T w2 = t.w[p0] * t.w[p1], td = tau_d[e] * t.vol * w2;
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = td * t.w[q] * (a0[s0 * q] + a1[s1 * q] + a2[s2 * q]);
    eo_apply<N, -1>(t.Dt, x, v);
#pragma unroll
    for (int r = 0; r < N; ++r) x[r] = fmadd(t.ih[j], v[r], mw[r]);
    eo_apply<N, 1>(t.St, x, v);
    v[0] += L[C::FC + 2 * j] * w2 * aj[0];
    v[N - 1] += L[C::FC + 2 * j + 1] * w2 * aj[SN * (N + 1)];
#pragma unroll
    for (int r = 0; r < N; ++r) mw[r] = v[r];
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int r = 0; r < N; ++r) aj[SN * (r + 1)] = mw[r];
  }
  __syncthreads();
  // ---- P4: S^T along t2
  if (active) {
    T* a = A + SN * (p1 + 1) + S1 * p0;
    T x[N], v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = a[q];
    eo_apply<N, 1>(fresh(tab)->St, x, v);
#pragma unroll
    for (int q = 0; q < N; ++q) a[q] = v[q];
  }
  __syncthreads();
  // ---- P5: S^T along t1, store; lanes run along x (n for j = 0, else t2)
  T acc = 0;   // this thread's part of u.y (dot only)
  if (active) {
    const T* a = A + SN + (j == 0 ? SN * p0 + p1 : p0 + SN * p1);
    T x[N], v[N];
#pragma unroll
    for (int c = 0; c < N; ++c) x[c] = a[S1 * c];
    eo_apply<N, 1>(fresh(tab)->St, x, v);
    const size_t o = j * cs + (size_t)e * N3 + p0 + (j == 2 ? N2 : N) * p1;
    const int gs = j == 2 ? N : N2;
#pragma unroll
    for (int c = 0; c < N; ++c) y[o + gs * c] = v[c];
    if (dot) {   // u.y of this pencil (the input again, from cache)
#pragma unroll
      for (int c = 0; c < N; ++c) acc = fmadd(u[o + gs * c], v[c], acc);
    }
  }
  // ---- optional: workgroup sum of u.y into dot[blockIdx.x] (fixed order)
  if (dot) {
    __syncthreads();
    lds[tid] = acc;
    __syncthreads();
    if (tid < 64) {   // one wavefront
      T s = 0;
      for (int i = tid; i < C::THREADS; i += 64) s += lds[i];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (tid == 0) dot[blockIdx.x] = s;
    }
  }
}

// Even-odd tables of the n x n row-major matrix A (parity sig); false if A
// lacks that parity.
template <int N, typename T>
bool make_eo(const double* A, int sig, EOMat<N, T>& m) {
  constexpr int H = N / 2;
  double amax = 0;
  for (int i = 0; i < N * N; ++i) amax = std::max(amax, std::fabs(A[i]));
  for (int i = 0; i < N; ++i)
    for (int k = 0; k < N; ++k)
      if (std::fabs(A[(N - 1 - i) * N + (N - 1 - k)] - sig * A[i * N + k]) > 1e-11 * amax) return false;
  for (int i = 0; i < H; ++i) {
    for (int k = 0; k < H; ++k) {
      m.P[i][k] = (T)(0.5 * (A[i * N + k] + A[i * N + N - 1 - k]));
      m.Q[i][k] = (T)(0.5 * (A[i * N + k] - A[i * N + N - 1 - k]));
    }
    m.col[i] = (T)(N % 2 ? A[i * N + H] : 0.0);
    m.row[i] = (T)(N % 2 ? A[H * N + i] : 0.0);
  }
  m.mid = (T)(N % 2 ? A[H * N + H] : 0.0);
  return true;
}

template <int N, typename T>
bool make_proj_tab(const ProjPlan& P, ProjTab<N, T>& t) {
  double St[N * N], Dt[N * N];
  for (int i = 0; i < N; ++i) {
    for (int a = 0; a < N; ++a) {
      St[a * N + i] = P.S[i * N + a];
      Dt[a * N + i] = P.Dg[i * N + a];
    }
    t.w[i] = (T)P.w[i];
  }
  if (!make_eo<N, T>(P.S.data(), 1, t.S) || !make_eo<N, T>(St, 1, t.St) || !make_eo<N, T>(P.Dg.data(), -1, t.Dg) ||
      !make_eo<N, T>(Dt, -1, t.Dt))
    return false;
  t.vol = (T)P.vol;
  for (int d = 0; d < 3; ++d) {
    t.ih[d] = (T)P.ih[d];
    t.area[d] = (T)P.area[d];
  }
  return true;
}

template <int N, typename T>
hipError_t launch_n(const ProjPlan& P, const void* u, void* yv, const void* td, const void* tc, hipStream_t s,
                    void* dot) {
  std::atomic<const void*>& slot = P.tab.p[sizeof(T) == 4];
  const ProjTab<N, T>* dt = static_cast<const ProjTab<N, T>*>(slot.load(std::memory_order_acquire));
  if (!dt) {
    ProjTab<N, T> t{};
    if (!make_proj_tab<N, T>(P, t)) return hipErrorInvalidValue;
    hipError_t err;
    if (!(dt = device_table_of("projection", t, &err))) return err;
    slot.store(dt, std::memory_order_release);
  }
  using C = ProjCfg<N>;
  const long long grid = ((long long)P.mesh.n_el + C::E - 1) / C::E;
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((projection_kernel<N, T>), dim3((unsigned)grid), dim3(C::THREADS), 0, s, (const T*)u,
                     (T*)yv, (const T*)td, (const T*)tc, P.mesh, dt, (T*)dot);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const ProjPlan& P, const void* u, void* y, const void* td, const void* tc, hipStream_t s,
                    void* dot) {
  switch (P.k) {
    case 1: return launch_n<2, T>(P, u, y, td, tc, s, dot);
    case 2: return launch_n<3, T>(P, u, y, td, tc, s, dot);
    case 3: return launch_n<4, T>(P, u, y, td, tc, s, dot);
    case 4: return launch_n<5, T>(P, u, y, td, tc, s, dot);
    case 5: return launch_n<6, T>(P, u, y, td, tc, s, dot);
    case 6: return launch_n<7, T>(P, u, y, td, tc, s, dot);
    case 7: return launch_n<8, T>(P, u, y, td, tc, s, dot);
    case 8: return launch_n<9, T>(P, u, y, td, tc, s, dot);
    case 9: return launch_n<10, T>(P, u, y, td, tc, s, dot);
    case 10: return launch_n<11, T>(P, u, y, td, tc, s, dot);
    case 11: return launch_n<12, T>(P, u, y, td, tc, s, dot);
    default: return hipErrorInvalidValue;
  }
}

template <int N>
long long grid_n(long long n_el) {
  return (n_el + ProjCfg<N>::E - 1) / ProjCfg<N>::E;
}

}  // namespace

hipError_t launch_projection(const ProjPlan& P, bool f32, const void* u, void* y, const void* tau_d,
                             const void* tau_c, hipStream_t s, void* dot_partial) {
  return f32 ? launch_t<float>(P, u, y, tau_d, tau_c, s, dot_partial)
             : launch_t<double>(P, u, y, tau_d, tau_c, s, dot_partial);
}

long long projection_grid(const ProjPlan& P) {
  const long long n = P.mesh.n_el;
  switch (P.k) {
    case 1: return grid_n<2>(n);
    case 2: return grid_n<3>(n);
    case 3: return grid_n<4>(n);
    case 4: return grid_n<5>(n);
    case 5: return grid_n<6>(n);
    case 6: return grid_n<7>(n);
    case 7: return grid_n<8>(n);
    case 8: return grid_n<9>(n);
    case 9: return grid_n<10>(n);
    case 10: return grid_n<11>(n);
    case 11: return grid_n<12>(n);
    default: return 0;
  }
}

}  // namespace dgmf
