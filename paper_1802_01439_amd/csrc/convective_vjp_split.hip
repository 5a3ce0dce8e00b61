// Vector-Jacobian product of the convective term (the form of
// convective_vjp.hip) with one thread per pencil AND velocity component, in
// passes over the derivative direction, FP64 k >= 2 and FP32 k >= 4 (but for
// two ranges of mesh sizes, see vjp_onepass).
//
//   P_k = sum_d [ c_d u_d d_d w_k + delta_kd c_d sum_c u_c d_d w_c ],
//
// so pass d needs, per thread, d_d w_k along its own pencil, u_d (from an LDS
// buffer that component d fills) and, for component d alone, the sum over the
// components of u_c d_d w_c, which the other two send through LDS.  A thread
// holds u_k and P_k at the m points and one pencil of n values: 64 to 143
// registers in FP64; k = 11, capped at 128 by its 14 wavefronts, spills 16 (68
// bytes a lane), and k = 6, 8, 9, 10 hold 7 to 30 scalar registers of table rows
// in vector lanes.  The kernels this one replaces held all four swept fields
// of u and w at once: 43 KB of LDS per element at k = 4, 155 KB at k = 11,
// where the registers spilled to memory (17 ms for 1.6e7 nodes).
// Sweep and data layout as in convective_split.hip; written here for z first
// and x pencils last (FP64), in FP32 x and z change places (see the launch).
//
//   z sweep of u (and of the x neighbours' facing layers); first sweep of the
//   y- and z-face lines of u (own, neighbour) and of w own - w neighbour |
//   y sweep of u; on the last wavefronts the face pencils (one component per
//   lane; the normal velocities and the sum for the normal component come
//   from the lanes that hold them) | x pencils of u, x-face coefficients |
//   per pass d = x, y, z:  z sweep of w (G for d = z), u_d to LDS |
//     y sweep (G for d = y) | x sweep (G for d = x), P_k, products out |
//     component d adds the products |
//   S^T_x | S^T_y (+ y faces) | S^T_z (+ z faces), write-out.
// w is read from memory in each pass (twice from the caches), one pass ahead.
//
// What bounds it: the vector ALU and the chain of 18 to 21 short phases.
// Measured, microseconds, against the kernels with three components per
// thread:  FP64 k = 2 (60^3) 620 -> 523, 3 (32^3) 162 -> 136, 4 (32^3) 510
// -> 286, 5 (28^3) 564 -> 257, 6 (24^3) 786 -> 370, 7 (20^3) 520 -> 314,
// 8 (18^3) 751 -> 277, 9 (16^3) 734 -> 352, 10 (15^3) 1189 -> 368,
// 11 (21^3) 17712 -> 1570; FP32 on the degree-sweep meshes k = 4 830 -> 661,
// 5 796 -> 524, 6 1093 -> 595, 7 740 -> 546, 8 920 -> 550, 9 1094 -> 672,
// 10 1799 -> 575, 11 1526 -> 799.  FP32 k = 2 (40^3) 75 -> 87 and k = 3 (32^3)
// 75 -> 77 us: those keep the one-pass kernel.
#include <cmath>
#include <type_traits>

#include "api_internal.h"
#include "common.h"
#include "conv_common.h"
#include "ops.h"

namespace dgmf {

// 1D tables in even-odd form (see ConvTab), the Gauss weights folded into S^T.
template <int N, int Q, typename T>
struct VjpTab {
  static constexpr int NH = N / 2, NC = (N + 1) / 2, QH = Q / 2, QC = (Q + 1) / 2;
  T Sp[QC][NH], Sm[QC][NH], Sc[QC];   // S, rows q < ceil(m/2)
  T Gp[QC][NH], Gm[QC][NH], Gc[QC];   // G, rows q < ceil(m/2)
  T Tp[QH][NC], Tm[QH][NC], Tc[NC];   // S^T W, by input pair q < m/2
};

template <int N, int Q, typename T>
constexpr VjpTab<N, Q, T> make_vjp_tab(const double* S, const double* G, const double* w) {
  using Tb = VjpTab<N, Q, T>;
  Tb t{};
  for (int q = 0; q < Tb::QC; ++q) {
    for (int a = 0; a < Tb::NH; ++a) {
      t.Sp[q][a] = (T)(0.5 * (S[q * N + a] + S[q * N + N - 1 - a]));
      t.Sm[q][a] = (T)(0.5 * (S[q * N + a] - S[q * N + N - 1 - a]));
      t.Gp[q][a] = (T)(0.5 * (G[q * N + a] + G[q * N + N - 1 - a]));
      t.Gm[q][a] = (T)(0.5 * (G[q * N + a] - G[q * N + N - 1 - a]));
    }
    t.Sc[q] = (N % 2) ? (T)S[q * N + Tb::NH] : T(0);
    t.Gc[q] = (N % 2) ? (T)G[q * N + Tb::NH] : T(0);
  }
  for (int q = 0; q < Tb::QH; ++q)
    for (int a = 0; a < Tb::NC; ++a) {
      const double h = 0.5 * w[q];
      t.Tp[q][a] = (T)(h * (S[q * N + a] + S[(Q - 1 - q) * N + a]));
      t.Tm[q][a] = (T)(h * (S[q * N + a] - S[(Q - 1 - q) * N + a]));
    }
  for (int a = 0; a < Tb::NC; ++a) t.Tc[a] = (Q % 2) ? (T)(w[Tb::QH] * S[Tb::QH * N + a]) : T(0);
  return t;
}

template <int N, int Q, typename T>
constexpr VjpTab<N, Q, T> vjp_tab_ct() {
  constexpr ct::Tables<N, Q> d{};
  double S[Q * N] = {}, G[Q * N] = {};
  for (int q = 0; q < Q; ++q)
    for (int a = 0; a < N; ++a) {
      S[q * N + a] = d.S[q][a];
      G[q * N + a] = d.G[q][a];
    }
  return make_vjp_tab<N, Q, T>(S, G, d.w);
}

template <int N, int Q, typename T>
__device__ __forceinline__ decltype(auto) vjp_pick(const VjpTab<N, Q, T>& ct, const VjpTab<N, Q, T>* tab) {
  if constexpr (sizeof(T) == 4) return (ct);
  else return *fresh(tab);
}

#define VJP_TABLES(t)                                             \
  constexpr VjpTab<N, Q, T> t##_ct =                              \
      sizeof(T) == 4 ? vjp_tab_ct<N, Q, T>() : VjpTab<N, Q, T>{}; \
  const auto& t = vjp_pick<N, Q, T>(t##_ct, tab)

// LDS layout of one element (units of T): slots, face layers and their
// pitches as in convective_split.hip, without that kernel's pads between the
// layers (they were counted for its phases, not for these).  UB: c_d u_d of the pass; before that
// (over the same space) the neighbour u layers and the w differences.
// A pencil's m products (and two x-face terms) for component d go to its own
// n+2 slots, which it has read by then, and m-n values beyond those: to extra
// column blocks, or, where these would cost a workgroup per CU (FP64 k = 8)
// or do not fit (FP64 k = 11), from registers to UB one phase later (LATE).
template <int N, int Q, int SZ>
struct VjpSplitShape {
  static constexpr int N2 = N * N, N3 = N * N * N;
  static constexpr int COLS = N == 5 ? 50 : (Q * Q) | 1;
  static constexpr int FP = N == 6 ? 9 : N == 11 ? 17 : Q;   // pitch of a face layer
  static constexpr int LAYER = N * FP;
  static constexpr int FL = 6 * LAYER;
  static constexpr bool LATE = SZ == 8 && (N == 9 || N == 12);
  static constexpr int NX = Q - N;
  static constexpr int UBo = 3 * (N + 2) * COLS;
  static constexpr int EXo = UBo + Q * COLS;
  static constexpr int UEND = EXo + (LATE ? 0 : 2 * NX * COLS);
  static constexpr int NBo = UBo;   // neighbour u layers, then w differences: dead before UB is filled
  static constexpr int FOo = UEND > NBo + 4 * FL ? UEND : NBo + 4 * FL;
  static constexpr int PER = FOo + 2 * FL;
  static constexpr int BYTES = PER * SZ;
  static constexpr int NW = (3 * Q * Q + 63) / 64, TH = NW * 64;
  // register caps where the count lies just above a step of the wavefronts per
  // SIMD: FP64 k = 6 481 -> 367 us (96 registers), k = 8 430 -> 276 (128)
  static constexpr int MINW = SZ == 8 && N == 7 ? 5 : SZ == 8 && N == 9 ? 4 : 1;
  static_assert(BYTES <= 160 * 1024, "VJP LDS footprint exceeds 160 KB");
  static_assert(!LATE || 2 * NX <= Q, "the late values fit the u buffer");
};

template <int N, int Q, typename T, int TH, int DA, int DC>
__global__ void __launch_bounds__(TH)
    __attribute__((amdgpu_waves_per_eu(VjpSplitShape<N, Q, (int)sizeof(T)>::MINW, 8)))
    vjp_split_kernel(const T* __restrict__ u, const T* __restrict__ wv, T* __restrict__ g, MeshArgs mesh,
                     const VjpTab<N, Q, T>* __restrict__ tab, ConvScal<T> sc) {
  using Sh = VjpSplitShape<N, Q, (int)sizeof(T)>;
  constexpr int N2 = Sh::N2, N3 = Sh::N3, COLS = Sh::COLS, SA = 3 * COLS;
  constexpr int LAYER = Sh::LAYER, FL = Sh::FL, FP = Sh::FP, NW = Sh::NW, NX = Sh::NX;
  constexpr int UBo = Sh::UBo, EXo = Sh::EXo, NBo = Sh::NBo, FOo = Sh::FOo;
  constexpr int NH = N / 2, QH = Q / 2, QQ = Q * Q;
  // strides between the nodes along DA (first sweep) and DC (pencils at the
  // Gauss points); the middle direction is y
  static_assert(DA + DC == 2 && DA != DC, "x and z in either order");
  constexpr int TA = DA ? N2 : 1, TC = DC ? N2 : 1;
  extern __shared__ double dyn_lds[];
  T* lds = reinterpret_cast<T*>(dyn_lds);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const size_t cs = (size_t)mesh.n_el * N3;
  const int nxy = mesh.nx * mesh.ny;
  const int el = xcd_remap(blockIdx.x, gridDim.x);
  const int ez = el / nxy, exy = el - ez * nxy, ey = exy / mesh.nx, ex = exy - ey * mesh.nx;

  // sweep of n values with S or G
  auto sweep = [&](auto grad, const T (&x)[N], auto&& st) {
    VJP_TABLES(t);
    if constexpr (decltype(grad)::value) eo_interp_g<N, Q, T>(t, x, st);
    else eo_interp<N, Q, T>(t, x, st);
  };
  // source and LDS slot of column item w < 3 n^2 (element) or of the x neighbours' facing layers (6 n more)
  auto column = [&](int w, const T* f, const T*& src, int& dst) {
    if (w < 3 * N2) {
      const int j = w / N2, ab = w - j * N2, b = ab / N, a = ab - b * N;
      src = f + j * cs + (size_t)el * N3 + TC * a + N * b;
      dst = (a + 1) * SA + j * COLS + Q * b;
    } else {
      const int v = w - 3 * N2, p = v % N, r1 = v / N, s = r1 & 1, j = r1 >> 1;
      src = f + j * cs + (size_t)neighbor(mesh, ex, ey, ez, DC, s) * N3 + (s ? 0 : TC * (N - 1)) + N * p;
      dst = (s ? N + 1 : 0) * SA + j * COLS + Q * p;
    }
  };

  // ---- z sweeps of u; first sweeps of the y- and z-face layers
  {
    constexpr int nC = 3 * N2 + 6 * N, total = nC + 36 * N, NI = (total + TH - 1) / TH;
    T in[NI][N];
    int d1[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int w = tid + i * TH;
      d1[i] = -1;
      if (w >= total) continue;
      if (w < nC) {
        const T* src;
        column(w, u, src, d1[i]);
#pragma unroll
        for (int c = 0; c < N; ++c) in[i][c] = src[TA * c];
      } else {   // type 0: u own, 1: u neighbour, 2: w own - w neighbour
        const int v = w - nC, p = v % N, r = v / N, fam = r / 18, r2 = r - fam * 18, type = r2 / 6, sj = r2 - type * 6;
        const int s = sj & 1, j = sj >> 1;
        const int nb = neighbor(mesh, ex, ey, ez, fam ? DA : 1, s);
        const int stride = fam ? N : TA, lstep = fam ? TA : N;   // along the line; between layers
        const size_t oown = (size_t)el * N3 + TC * p + lstep * (s ? N - 1 : 0);
        const size_t onb = (size_t)nb * N3 + TC * p + lstep * (s ? 0 : N - 1);
        const T* f = (type == 2 ? wv : u) + j * cs;
        const T* src = f + (type == 1 ? onb : oown);
#pragma unroll
        for (int c = 0; c < N; ++c) in[i][c] = src[c * stride];
        if (type == 2) {
          const T* sn = f + onb;
#pragma unroll
          for (int c = 0; c < N; ++c) in[i][c] -= sn[c * stride];
        }
        d1[i] = (type == 0 ? FOo : NBo + (type - 1) * 2 * FL) + fam * FL + (3 * s + j) * LAYER + p * FP;
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (d1[i] < 0) continue;
      T* p = lds + d1[i];
      sweep(std::false_type{}, in[i], [&](int q, T v) { p[q] = v; });
    }
  }
  lds_barrier();

  // y sweep in place of the x layers [a0, a1)
  auto y_sweep = [&](auto grad, int a0, int a1) {
    const int nl = a1 - a0;
    for (int w = tid; w < 3 * nl * Q; w += TH) {
      const int q3 = w % Q, rest = w / Q, j = rest % 3, al = a0 + rest / 3;
      T* p = lds + al * SA + j * COLS + q3;
      T x[N];
#pragma unroll
      for (int b = 0; b < N; ++b) x[b] = p[Q * b];
      sweep(grad, x, [&](int q, T v) { p[Q * q] = v; });
    }
  };

  // adjoint flux coefficients at a face point: own/neighbour normal velocity
  // (times the outward sign) unm, unp and own/neighbour values um, up of the
  // thread's component: dw_k enters G_k with diag and the normal component's
  // G with ex
  auto adj = [&](T sgn, T unm, T unp, T um, T up, T& diag, T& exk) {
    const T am = fabs(unm), ap = fabs(unp), lam = fmax(am, ap);
    const T sm = am > ap ? T(1) : (am == ap ? T(0.5) : T(0));
    const T sgu = unm > T(0) ? T(1) : (unm < T(0) ? T(-1) : T(0));
    diag = T(0.5) * unm + sc.lf * lam;
    exk = sgn * (T(0.5) * um + sc.lf * sm * sgu * (um - up));
  };

  // ---- y sweep of u; y- and z-face pencils on the last wavefronts
  {
    constexpr int FT = (4 * Q + 20) / 21;
    static_assert(FT <= NW, "one round of face pencils");
    if (wave >= NW - FT) {
      const int j = lane / 21, i21 = lane - 21 * j, fc = (NW - 1 - wave) * 21 + i21;
      if (lane < 63 && fc < 4 * Q) {
        const int fam = fc / (2 * Q), rem = fc - fam * 2 * Q, s = rem / Q, q = rem - s * Q;
        const int fo = fam * FL + (3 * s + j) * LAYER + q;
        T* F = lds + FOo + fo;
        const T* Fn = lds + NBo + fo;
        const T* Fw = Fn + 2 * FL;
        const int nj = fam ? DA : 1, nl = (i21 + 21 * nj) * 4;   // normal component and its lane
        const int l1 = (i21 + 21 * ((j + 1) % 3)) * 4, l2 = (i21 + 21 * ((j + 2) % 3)) * 4;
        VJP_TABLES(t);
        // even-odd parts of the lines u own, u neighbour, dw; those of dw are
        // formed again for each point pair where they would not fit in the
        // registers (FP64 k = 11)
        constexpr bool AGAIN = sizeof(T) == 8 && N == 12;
        T xe[3][NH], xo[3][NH], xm[3];
        auto split = [&](const T* src, int f) {
          T x[N];
#pragma unroll
          for (int c = 0; c < N; ++c) x[c] = src[c * FP];
#pragma unroll
          for (int a = 0; a < NH; ++a) {
            xe[f][a] = x[a] + x[N - 1 - a];
            xo[f][a] = x[a] - x[N - 1 - a];
          }
          xm[f] = (N % 2) ? x[NH] : T(0);
        };
        split(F, 0);
        split(Fn, 1);
        if constexpr (!AGAIN) split(Fw, 2);
        EoT<N, T, 1> acc;
        acc.zero();
        const T sgn = s ? T(1) : T(-1);
        const T wgt = fam ? sc.area[DA] : sc.area[1];
        auto point = [&](T um, T up, T dw) {
          const T unm = sgn * lane_get(nl, um), unp = sgn * lane_get(nl, up);
          T diag, exk;
          adj(sgn, unm, unp, um, up, diag, exk);
          const T e = exk * dw;
          const T e1 = lane_get(l1, e), e2 = lane_get(l2, e);
          return wgt * (dw * diag + (j == nj ? e + e1 + e2 : T(0)));
        };
#pragma unroll
        for (int q1 = 0; q1 < (Q + 1) / 2; ++q1) {
          T ev[3], ov[3];
          if constexpr (AGAIN) {
            int off = fo;
            asm volatile("" : "+v"(off));
            split(lds + NBo + 2 * FL + off, 2);
          }
#pragma unroll
          for (int f = 0; f < 3; ++f) {
            ev[f] = t.Sp[q1][0] * xe[f][0];
            ov[f] = t.Sm[q1][0] * xo[f][0];
#pragma unroll
            for (int a = 1; a < NH; ++a) {
              ev[f] = fmadd(t.Sp[q1][a], xe[f][a], ev[f]);
              ov[f] = fmadd(t.Sm[q1][a], xo[f][a], ov[f]);
            }
            if constexpr (N % 2 == 1) ev[f] = fmadd(t.Sc[q1], xm[f], ev[f]);
          }
          const T gq = point(ev[0] + ov[0], ev[1] + ov[1], ev[2] + ov[2]);
          if (q1 < QH) {
            const T gr = point(ev[0] - ov[0], ev[1] - ov[1], ev[2] - ov[2]);
            acc.pair(t.Tp[q1], t.Tm[q1], gq, gr);
          } else {
            acc.mid(t.Tc, gq);
          }
        }
#pragma unroll
        for (int c = 0; c < N; ++c) F[c * FP] = acc.out(c);
      }
    }
    y_sweep(std::false_type{}, 0, N + 2);
  }
  lds_barrier();

  // columns of w, loaded one pass ahead
  constexpr int nW = 3 * N2 + 6 * N;
  static_assert(nW <= TH, "one column of w per thread");
  T win[N];
  int wdst = -1;
  auto issue_w = [&](int count) {
    wdst = -1;
    if (tid < count) {
      const T* src;
      column(tid, wv, src, wdst);
#pragma unroll
      for (int c = 0; c < N; ++c) win[c] = src[TA * c];
    }
  };
  issue_w(nW);

  // ---- x pencils of u, items (j, q2, q3)
  const int j3 = tid / QQ, qq = tid - j3 * QQ;
  const bool own = tid < 3 * QQ;
  T* colb = lds + (own ? qq : 0);
  T* col = colb + (own ? j3 * COLS : 0);
  T* buf = colb + UBo;
  T U[Q], P[Q];
  T dg0 = 0, dg1 = 0, ex0 = 0, ex1 = 0, F0 = 0, F1 = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) P[q] = T(0);
  if (own) {
    T x[N];
    const T vL = col[0], vR = col[(N + 1) * SA];
#pragma unroll
    for (int c = 0; c < N; ++c) x[c] = col[(c + 1) * SA];
    const T* cn = colb + DC * COLS;   // normal component
    adj(T(-1), -cn[SA], -cn[0], x[0], vL, dg0, ex0);
    adj(T(1), cn[N * SA], cn[(N + 1) * SA], x[N - 1], vR, dg1, ex1);
    sweep(std::false_type{}, x, [&](int q, T v) { U[q] = v; });
  }
  lds_barrier();

  // ---- passes over the derivative direction d
  auto pass = [&](auto dc) {
    constexpr int d = decltype(dc)::value;
    using GA = std::integral_constant<bool, d == DA>;
    using GB = std::integral_constant<bool, d == 1>;
    using GC = std::integral_constant<bool, d == DC>;
    const T cd = sc.cell[d];
    if (wdst >= 0) {
      T* p = lds + wdst;
      sweep(GA{}, win, [&](int q, T v) { p[q] = v; });
    }
    if (own && j3 == d) {
#pragma unroll
      for (int q = 0; q < Q; ++q) buf[q * COLS] = cd * U[q];
    }
    lds_barrier();
    if constexpr (d == DC) y_sweep(GB{}, 0, N + 2);
    else y_sweep(GB{}, 1, N + 1);
    lds_barrier();
    T late[NX];
    const int which = (j3 - d + 3) % 3 - 1;   // -1: component d itself
    T* ext = colb + (Sh::LATE ? UBo : EXo) + (which > 0 ? NX * COLS : 0);
    // value i < m + 2 sent to component d: the product at point i, then the x-face terms
    auto put = [&](int i, T v) {
      if (i < N + 2) col[i * SA] = v;
      else if constexpr (Sh::LATE) late[i - N - 2] = v;
      else ext[(i - N - 2) * COLS] = v;
    };
    if (own) {
      T x[N];
#pragma unroll
      for (int c = 0; c < N; ++c) x[c] = col[(c + 1) * SA];
      T e0 = 0, e1 = 0;
      if constexpr (d == DC) {
        const T dw0 = x[0] - col[0], dw1 = x[N - 1] - col[(N + 1) * SA];
        F0 = sc.area[DC] * (dw0 * dg0);
        F1 = sc.area[DC] * (dw1 * dg1);
        e0 = sc.area[DC] * (dw0 * ex0);
        e1 = sc.area[DC] * (dw1 * ex1);
      }
      if (which < 0) {
        sweep(GC{}, x, [&](int q, T v) { P[q] = fmadd(T(2) * buf[q * COLS], v, P[q]); });
        F0 += e0;
        F1 += e1;
      } else {
        sweep(GC{}, x, [&](int q, T v) {
          P[q] = fmadd(buf[q * COLS], v, P[q]);
          put(q, U[q] * v);
        });
        if constexpr (d == DC) {
          put(Q, e0);
          put(Q + 1, e1);
        }
      }
    }
    if constexpr (d != DA && !Sh::LATE) issue_w(3 * N2);
    lds_barrier();
    if constexpr (Sh::LATE) {
      if (own && which >= 0) {
#pragma unroll
        for (int i = 0; i < NX; ++i) ext[i * COLS] = late[i];
      }
      if constexpr (d != DA) issue_w(3 * N2);
      lds_barrier();
    }
    if (own && which < 0) {
      const T *c1 = colb + ((d + 1) % 3) * COLS, *c2 = colb + ((d + 2) % 3) * COLS;
      const T *x1 = colb + (Sh::LATE ? UBo : EXo), *x2 = x1 + NX * COLS;
      auto get = [&](int i) { return i < N + 2 ? c1[i * SA] + c2[i * SA] : x1[(i - N - 2) * COLS] + x2[(i - N - 2) * COLS]; };
#pragma unroll
      for (int q = 0; q < Q; ++q) P[q] = fmadd(cd, get(q), P[q]);
      if constexpr (d == DC) {
        F0 += get(Q);
        F1 += get(Q + 1);
      }
    }
    lds_barrier();
  };
  pass(std::integral_constant<int, DC>{});
  pass(std::integral_constant<int, 1>{});
  pass(std::integral_constant<int, DA>{});

  // ---- back sweeps
  auto back = [&](EoT<N, T, 1>& a, auto&& val) {
    VJP_TABLES(t);
    a.zero();
#pragma unroll
    for (int q = 0; q < QH; ++q) a.pair(t.Tp[q], t.Tm[q], val(q), val(Q - 1 - q));
    if constexpr (Q % 2 == 1) a.mid(t.Tc, val(QH));
  };
  if (own) {
    EoT<N, T, 1> a;
    back(a, [&](int q) { return P[q]; });
#pragma unroll
    for (int c = 0; c < N; ++c) {
      T o = a.out(c);
      if (c == 0) o += F0;
      if (c == N - 1) o += F1;
      col[c * SA] = o;
    }
  }
  lds_barrier();
  constexpr int nY = 3 * N * Q, nZ = 3 * N2;
  if (tid < nY) {
    const int q3 = tid % Q, rest = tid / Q, a0 = rest % N, j = rest / N;
    T* p = lds + a0 * SA + j * COLS + q3;
    EoT<N, T, 1> a;
    back(a, [&](int q) { return p[Q * q]; });
    const T* F = lds + FOo + j * LAYER + a0 * FP + q3;
    const T f0 = F[0], f1 = F[3 * LAYER];
#pragma unroll
    for (int b = 0; b < N; ++b) p[Q * b] = a.out(b) + (b == 0 ? f0 : T(0)) + (b == N - 1 ? f1 : T(0));
  }
  {   // z-face terms: integrate in y, in place
    constexpr int nF = 6 * N, FI = wave_split(nY, nF, TH);
    for (int w = tid; w < FI + nF; w += TH) {
      if (w < FI) continue;
      const int v = w - FI, sj = v / N;   // sj = 3 s + j
      T* F = lds + FOo + FL + sj * LAYER + (v - sj * N) * FP;
      EoT<N, T, 1> a;
      back(a, [&](int q) { return F[q]; });
#pragma unroll
      for (int b = 0; b < N; ++b) F[b] = a.out(b);
    }
  }
  lds_barrier();
  if (tid < nZ) {
    const int j = tid / N2, ab = tid - j * N2, b = ab / N, a0 = ab - b * N;
    const T* p = lds + a0 * SA + j * COLS + Q * b;
    EoT<N, T, 1> a;
    back(a, [&](int q) { return p[q]; });
    const T* F = lds + FOo + FL + j * LAYER + a0 * FP + b;
    const T f0 = F[0], f1 = F[3 * LAYER];
    T* out = g + j * cs + (size_t)el * N3 + TC * a0 + N * b;
#pragma unroll
    for (int c = 0; c < N; ++c) out[TA * c] = a.out(c) + (c == 0 ? f0 : T(0)) + (c == N - 1 ? f1 : T(0));
  }
}

template <int N, int Q, typename T>
static hipError_t launch_vjp_split_nq(const ConvPlan& P, const void* u, const void* w, void* g, hipStream_t s) {
  using Sh = VjpSplitShape<N, Q, (int)sizeof(T)>;
  if (!conv_tables_match<N, Q>(P)) return hipErrorInvalidValue;
  ConvScal<T> sc;
  for (int d = 0; d < 3; ++d) {
    sc.cell[d] = (T)P.cell[d];
    sc.area[d] = (T)P.area[d];
  }
  sc.lf = (T)P.lf;
  const VjpTab<N, Q, T>* dt = nullptr;   // FP32 kernels use the compile-time tables
  if (sizeof(T) == 8) {
    hipError_t err;
    dt = plan_table<VjpTab<N, Q, T>>(
        P.tab.p[1], "vjp_split", [&] { return make_vjp_tab<N, Q, T>(P.S.data(), P.G.data(), P.w.data()); }, &err);
    if (!dt) return err;
  }
  // FP64: z first, so that a wavefront's loads and stores are contiguous.
  // FP32: x first.  The derivative of max(|u-.n|, |u+.n|) jumps where the two
  // are equal; the traces are rounded, so points closer to a tie than that
  // may fall on either side.  In this order the traces are formed as in the
  // one-pass kernel, bit for bit, and all FP32 degrees share its decisions.
  constexpr int DA = sizeof(T) == 4 ? 0 : 2;
  hipLaunchKernelGGL((vjp_split_kernel<N, Q, T, Sh::TH, DA, 2 - DA>), dim3(P.mesh.n_el), dim3(Sh::TH), Sh::BYTES, s, (const T*)u,
                     (const T*)w, (T*)g, P.mesh, dt, sc);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_vjp_split_t(const ConvPlan& P, const void* u, const void* w, void* g, hipStream_t s) {
  if constexpr (sizeof(T) == 8) {
    if (P.k == 2) return launch_vjp_split_nq<3, 4, T>(P, u, w, g, s);
    if (P.k == 3) return launch_vjp_split_nq<4, 5, T>(P, u, w, g, s);
  }
  switch (P.k) {
    case 4: return launch_vjp_split_nq<5, 7, T>(P, u, w, g, s);
    case 5: return launch_vjp_split_nq<6, 8, T>(P, u, w, g, s);
    case 6: return launch_vjp_split_nq<7, 10, T>(P, u, w, g, s);
    case 7: return launch_vjp_split_nq<8, 11, T>(P, u, w, g, s);
    case 8: return launch_vjp_split_nq<9, 13, T>(P, u, w, g, s);
    case 9: return launch_vjp_split_nq<10, 14, T>(P, u, w, g, s);
    case 10: return launch_vjp_split_nq<11, 16, T>(P, u, w, g, s);
    case 11: return launch_vjp_split_nq<12, 17, T>(P, u, w, g, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_convective_vjp_split(const ConvPlan& P, bool f32, const void* u, const void* w, void* g,
                                       hipStream_t s) {
  return f32 ? launch_vjp_split_t<float>(P, u, w, g, s) : launch_vjp_split_t<double>(P, u, w, g, s);
}

}  // namespace dgmf
