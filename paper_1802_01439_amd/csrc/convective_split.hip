// Convective term c_h (the form and the sweeps described in convective.hip)
// with one thread per pencil AND velocity component, for the degrees where
// one element fills several wavefronts: FP64 and FP32 from k = 4 on.
//
// What bounds this kernel and why the work is split so.  A thread that holds a
// whole pencil of all three components needs 200 to 256 registers in FP64:
// two wavefronts per SIMD, each with a serial chain of eleven phases, and the
// vector ALU is busy 32-50 % of the time.  Here a thread holds one component
// (m values) and one accumulator of n values at a time: 60 to 131 registers
// and nothing spilled to memory (FP64 k = 10 holds 144 scalar registers of
// table rows in vector lanes, k = 9 28, k = 11 21, k = 4, 6 and 8 two or three).  The back sweeps run in three passes over the flux direction
// f, in each of which all three components' threads work, instead of in
// three passes over the components.  The only thing the components exchange is
// u_f at the Gauss points of the pass, F_jf = u_j u_f, through an LDS buffer
// (m column blocks; ds_bpermute instead of the buffer costs 6.4 LDS cycles per
// 32-bit value, three times the write and reads of the buffer).
// Directions: the first sweep runs along z, so that a wavefront's loads and
// stores of the element block are contiguous; the pencils at the Gauss points
// run along x.  The Gauss weights are part of the back sweep tables.
//
//   P1  z sweeps of the element's columns, of the x neighbours' facing layers
//       (two extra x layers) and of the y neighbours' facing layers; y sweeps
//       of the own and neighbour z-face layers.  From global memory, all loads
//       first.
//   P2  y sweep in place (n+2 x layers); copies the own y-face layers out.
//   P3  x pencils: u_j at the m points into registers, the x-face fluxes; on
//       the last wavefronts the y- and z-face pencils (one component per
//       lane, 21 pencils per wavefront; a lane takes the normal component
//       from the lane that holds it).
//   pass f = x: G^T_x F_x | S^T_y, kept in registers (+ y faces)
//   pass f = y: S^T_x F_y | G^T_y, added, in place | S^T_z, kept (+ z faces)
//   pass f = z: S^T_x F_z | S^T_y in place | G^T_z, added, written out
// FP64 k >= 9 (one workgroup fills a CU's LDS) runs in persistent form: one
// workgroup per CU walks its share of the elements and loads the next element
// during the last pass.
//
// Measured on the degree-sweep meshes (about 1.7e7 nodes), microseconds,
// against the kernel with three components per thread:
//   FP64  k = 4 734 -> 638, 5 618 -> 544, 6 872 -> 676, 7 900 -> 629,
//         8 829 -> 614, 9 1306 -> 857, 10 1127 -> 817, 11 1183 -> 721
//   FP32  k = 4 425 -> 382, 5 377 -> 306, 6 393 -> 353, 7 327 -> 304,
//         8 367 -> 307, 9 406 -> 366, 10 433 -> 343, 11 430 -> 356
// and on 16^3 elements, FP64 k = 5: 38 -> 32.  Below k = 4 the kernel of
// convective.hip is faster (FP64 k = 3, 48^3: 240 against 247 us; FP32 142
// against 156).  The vector ALU is now busy 43-75 % of the time (FP64; 32-50 %
// before) resp. 92-100 % (FP32; four cycles per instruction), the LDS pipe
// 28-58 % resp. 56-80 % (four cycles per instruction and the conflicts).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "api_internal.h"
#include "common.h"
#include "conv_common.h"
#include "ops.h"

namespace dgmf {

// 1D tables in even-odd form (see ConvTab); the Gauss weights are folded into
// the transposed ones (they are symmetric too).
template <int N, int Q, typename T>
struct SplitTab {
  static constexpr int NH = N / 2, NC = (N + 1) / 2, QH = Q / 2, QC = (Q + 1) / 2;
  T Sp[QC][NH], Sm[QC][NH], Sc[QC];   // S, rows q < ceil(m/2)
  T Tp[QH][NC], Tm[QH][NC], Tc[NC];   // S^T W, by input pair q < m/2
  T Hp[QH][NC], Hm[QH][NC], Hc[NC];   // G^T W, by input pair q < m/2
};

template <int N, int Q, typename T>
constexpr SplitTab<N, Q, T> make_split_tab(const double* S, const double* G, const double* w) {
  using Tb = SplitTab<N, Q, T>;
  Tb t{};
  for (int q = 0; q < Tb::QC; ++q) {
    for (int a = 0; a < Tb::NH; ++a) {
      t.Sp[q][a] = (T)(0.5 * (S[q * N + a] + S[q * N + N - 1 - a]));
      t.Sm[q][a] = (T)(0.5 * (S[q * N + a] - S[q * N + N - 1 - a]));
    }
    t.Sc[q] = (N % 2) ? (T)S[q * N + Tb::NH] : T(0);
  }
  for (int q = 0; q < Tb::QH; ++q)
    for (int a = 0; a < Tb::NC; ++a) {
      const double h = 0.5 * w[q];
      t.Tp[q][a] = (T)(h * (S[q * N + a] + S[(Q - 1 - q) * N + a]));
      t.Tm[q][a] = (T)(h * (S[q * N + a] - S[(Q - 1 - q) * N + a]));
      t.Hp[q][a] = (T)(h * (G[q * N + a] + G[(Q - 1 - q) * N + a]));
      t.Hm[q][a] = (T)(h * (G[q * N + a] - G[(Q - 1 - q) * N + a]));
    }
  for (int a = 0; a < Tb::NC; ++a) {
    t.Tc[a] = (Q % 2) ? (T)(w[Tb::QH] * S[Tb::QH * N + a]) : T(0);
    t.Hc[a] = (Q % 2) ? (T)(w[Tb::QH] * G[Tb::QH * N + a]) : T(0);
  }
  return t;
}

template <int N, int Q, typename T>
constexpr SplitTab<N, Q, T> split_tab_ct() {
  constexpr ct::Tables<N, Q> d{};
  double S[Q * N] = {}, G[Q * N] = {};
  for (int q = 0; q < Q; ++q)
    for (int a = 0; a < N; ++a) {
      S[q * N + a] = d.S[q][a];
      G[q * N + a] = d.G[q][a];
    }
  return make_split_tab<N, Q, T>(S, G, d.w);
}

// FP32: compile-time constants; FP64: a device table read afresh in each
// phase (see conv_pick).
template <int N, int Q, typename T>
__device__ __forceinline__ decltype(auto) split_pick(const SplitTab<N, Q, T>& ct, const SplitTab<N, Q, T>* tab) {
  if constexpr (sizeof(T) == 4) return (ct);
  else return *fresh(tab);
}

#define SPLIT_TABLES(t)                                               \
  constexpr SplitTab<N, Q, T> t##_ct =                                \
      sizeof(T) == 4 ? split_tab_ct<N, Q, T>() : SplitTab<N, Q, T>{}; \
  const auto& t = split_pick<N, Q, T>(t##_ct, tab)

// LDS layout of one element (units of T).
//  Slots: slot a*3 + j is a column block of component j.  Forward: a = 0..n+1
//   are the x layers -1..n, entry (b, q3), after P2 (q2, q3), at q3 + m b.
//   Backward: a = 0..n-1 is the x node of the pass's back sweep.
//  U buffer (m column blocks, u_f of the current pass): over slots n, n+1 and
//   the neighbour face layers, which are dead by then.
//  Face layers NB (neighbour) and FO (own, then the pencils' results), each
//   y faces then z faces, [s][j][a][q], q = q3 (y faces) or q2 (z faces).
//  Pitches of the face layers and of the column blocks: chosen by counting,
//  for every phase, how many lanes of a half wavefront fall on each of the 32
//  8-byte banks, over pitches m and m + 1 and pads up to 16 (k = 5: a pitch of 9
//  instead of 8 and the pads below took the kernel from 563 to 544 us; k = 10
//  from 878 to 827).
template <int N, int Q, int SZ>
struct SplitShape {
  static constexpr int N2 = N * N, N3 = N * N * N;
  static constexpr int COLS = N == 5 ? 50 : (Q * Q) | 1;
  static constexpr int FP = N == 6 ? 9 : N == 11 ? 17 : Q;   // pitch of a face layer
  static constexpr int LAYER =
      N * FP + (N == 6 || N == 8 ? 2 : N == 7 ? 1 : N == 10 ? 3 : N == 12 ? 6 : 0);
  static constexpr int FL = 6 * LAYER + (N == 5 ? 1 : N == 6 ? 2 : N == 9 ? 4 : N == 10 ? 8 : 0);
  static constexpr int UBo = 3 * N * COLS;
  static constexpr int NBo = 3 * (N + 2) * COLS;
  static constexpr int FOo = NBo + 2 * FL > UBo + Q * COLS ? NBo + 2 * FL : UBo + Q * COLS;
  static constexpr int PER = FOo + 2 * FL;
  static constexpr int BYTES = PER * SZ;
  static constexpr int NW = (3 * Q * Q + 63) / 64, TH = NW * 64;
  // one workgroup per CU (k = 9 needs 84.4 KB, 3 % too much for two; k = 10 and
  // 11 119 and 143 KB): persistent form (FP64 k = 9 946 -> 857 us, k = 10
  // 820 -> 817, k = 11 763 -> 721).  Where more than one workgroup fits they
  // already hide each other's loads, and the registers of the loads in flight
  // cost a wavefront (k = 7 645 -> 736 us, FP32 k = 9 369 -> 415).
  static constexpr bool PERS = BYTES > 80 * 1024;
  // minimum wavefronts per SIMD (register cap).  The workgroups have 3 to 14
  // wavefronts and land on the SIMDs as they come, so full occupancy needs
  // room for an uneven spread: FP64 k = 6 (5 wavefronts) 802 -> 676 us at
  // <= 96 registers; FP32 k = 11 464 -> 358 us at 64
  static constexpr int MINW = SZ == 8 ? (N <= 6 ? 7 : N <= 8 ? 5 : N == 10 || N == 11 ? 3 : 4)
                                      : (N == 11 ? 7 : 8);
  static_assert(BYTES <= 160 * 1024, "convective LDS footprint exceeds 160 KB");
};

template <int N, int Q, typename T, int TH, bool PERS>
__global__ void __launch_bounds__(TH)
    __attribute__((amdgpu_waves_per_eu(SplitShape<N, Q, (int)sizeof(T)>::MINW, 8)))
    convective_split_kernel(const T* __restrict__ u, T* __restrict__ r, MeshArgs mesh,
                            const SplitTab<N, Q, T>* __restrict__ tab, ConvScal<T> sc) {
  using Sh = SplitShape<N, Q, (int)sizeof(T)>;
  constexpr int N2 = Sh::N2, N3 = Sh::N3, COLS = Sh::COLS, SA = 3 * COLS;
  constexpr int LAYER = Sh::LAYER, FL = Sh::FL, FP = Sh::FP, NW = Sh::NW;
  constexpr int UBo = Sh::UBo, NBo = Sh::NBo, FOo = Sh::FOo;
  constexpr int NH = N / 2, QH = Q / 2, QQ = Q * Q;
  // dynamic, so that the register cap is not overruled by the LDS size
  extern __shared__ double dyn_lds[];
  T* lds = reinterpret_cast<T*>(dyn_lds);
  // in the persistent form opaque to the compiler and taken afresh for each
  // element: otherwise every phase's index arithmetic is hoisted out of the
  // element loop and held in registers throughout
  auto thread_index = []() {
    int t = threadIdx.x;
    if constexpr (PERS) {
      asm volatile("" : "+v"(t));
      __builtin_assume(t >= 0 && t < TH);
    }
    return t;
  };
  auto bar = []() {
    if constexpr (PERS) lds_barrier();   // keeps the next element's loads in flight
    else __syncthreads();
  };
  const size_t cs = (size_t)mesh.n_el * N3;
  const int nxy = mesh.nx * mesh.ny;
  // elements of this workgroup: one, or in the persistent form every step-th
  // element of its XCD's contiguous share (workgroups go round-robin to the 8
  // XCDs; a grid of fewer than 8 splits the elements among as many shares)
  int el, eend, estep;
  if constexpr (PERS) {
    const int G = gridDim.x, x = blockIdx.x & 7, nx = G < 8 ? G : 8;
    estep = (G >> 3) + (x < (G & 7) ? 1 : 0);
    const int share = mesh.n_el / nx, more = mesh.n_el - share * nx;   // the first `more` XCDs take one more
    el = x * share + (x < more ? x : more);
    eend = el + share + (x < more ? 1 : 0);
    el += blockIdx.x >> 3;
  } else {
    el = xcd_remap(blockIdx.x, gridDim.x);
    eend = el + 1;
    estep = 1;
  }

  // ---- P1 loads: one pencil of one component per item
  constexpr int nM = 3 * N2, nL = 12 * N, nA = 12 * N;   // cell, x/y neighbour layers, z-face layers
  constexpr int total = nM + nL + nA;
  constexpr int NI = (total + TH - 1) / TH;
  T in[NI][N];
  int d1[NI];   // LDS destination, -1: no item
  auto issue = [&](int e0, bool live) {
    const int tid = thread_index();
    const int ez = e0 / nxy, exy = e0 - ez * nxy, ey = exy / mesh.nx, ex = exy - ey * mesh.nx;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int w = tid + i * TH;
      d1[i] = -1;
      const T* src = u;
      int stride = N2;
      if (live && w < total) {
        if (w < nM) {   // column (a, b)
          const int j = w / N2, ab = w - j * N2, b = ab / N, a = ab - b * N;
          src = u + j * cs + (size_t)e0 * N3 + ab;
          d1[i] = (a + 1) * SA + j * COLS + Q * b;
        } else if (w < nM + nL) {   // facing layer of an x or y neighbour
          const int v = w - nM, p = v % N, r1 = v / N;
          const int s = r1 & 1, r2 = r1 >> 1, j = r2 % 3, isy = r2 / 3;
          const int nb = neighbor(mesh, ex, ey, ez, isy, s), lay = s ? 0 : N - 1;
          src = u + j * cs + (size_t)nb * N3 + (isy ? p + N * lay : lay + N * p);
          d1[i] = isy ? NBo + (3 * s + j) * LAYER + p * FP : (s ? N + 1 : 0) * SA + j * COLS + Q * p;
        } else {   // z-face layer, own (sg 0) or neighbour, swept in y
          const int v = w - nM - nL, a = v % N, r1 = v / N;
          const int s = r1 & 1, r2 = r1 >> 1, sg = r2 & 1, j = r2 >> 1;
          const int e = sg ? neighbor(mesh, ex, ey, ez, 2, s) : e0;
          src = u + j * cs + (size_t)e * N3 + a + N2 * ((s != 0) != (sg != 0) ? N - 1 : 0);
          stride = N;
          d1[i] = (sg ? NBo : FOo) + FL + (3 * s + j) * LAYER + a * FP;
        }
      }
      if (d1[i] >= 0) {
#pragma unroll
        for (int c = 0; c < N; ++c) in[i][c] = src[c * stride];
      } else if constexpr (PERS) {
#pragma unroll
        for (int c = 0; c < N; ++c) in[i][c] = T(0);
      }
    }
  };

  issue(el, el < eend);
  for (; el < eend; el += estep) {
    const int tid = thread_index();
    const int wave = tid >> 6, lane = tid & 63;
    // ---- P1 sweeps
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (d1[i] >= 0) {
        SPLIT_TABLES(t);
        T* p = lds + d1[i];
        eo_interp<N, Q, T>(t, in[i], [&](int q, T v) { p[q] = v; });
      }
    }
    bar();

    // ---- P2: y sweep in place, items (j, x layer, q3)
    for (int w = tid; w < 3 * (N + 2) * Q; w += TH) {
      const int q3 = w % Q, rest = w / Q, al = rest % (N + 2), j = rest / (N + 2);
      SPLIT_TABLES(t);
      T* p = lds + al * SA + j * COLS + q3;
      T x[N];
#pragma unroll
      for (int b = 0; b < N; ++b) x[b] = p[Q * b];
      if (al >= 1 && al <= N) {   // own y-face layers, swept in z only
        T* F = lds + FOo + j * LAYER + (al - 1) * FP + q3;
        F[0] = x[0];
        F[3 * LAYER] = x[N - 1];
      }
      eo_interp<N, Q, T>(t, x, [&](int q, T v) { p[Q * q] = v; });
    }
    bar();

    // ---- P3: y- and z-face pencils (fam 0, 1), items (fam, s, q) x component, on
    // the last wavefronts: x sweep of both traces, flux at the m points, S^T_x
    constexpr int FT = (4 * Q + 20) / 21;   // wavefronts of 21 pencils
    static_assert(FT <= NW, "one round of face pencils");
    if (wave >= NW - FT) {
      const int j = lane / 21, i21 = lane - 21 * j, fc = (NW - 1 - wave) * 21 + i21;
      if (lane < 63 && fc < 4 * Q) {
        const int fam = fc / (2 * Q), rem = fc - fam * 2 * Q, s = rem / Q, q = rem - s * Q;
        SPLIT_TABLES(t);
        const int fo = fam * FL + (3 * s + j) * LAYER + q;
        T* F = lds + FOo + fo;
        const T* Fn = lds + NBo + fo;
        const int nl = (i21 + 21 * (fam + 1)) * 4;   // the lane of the normal component
        T xe[2][NH], xo[2][NH], xm[2];
#pragma unroll
        for (int sg = 0; sg < 2; ++sg) {
          T x[N];
#pragma unroll
          for (int c = 0; c < N; ++c) x[c] = sg ? Fn[c * FP] : F[c * FP];
#pragma unroll
          for (int a = 0; a < NH; ++a) {
            xe[sg][a] = x[a] + x[N - 1 - a];
            xo[sg][a] = x[a] - x[N - 1 - a];
          }
          xm[sg] = (N % 2) ? x[NH] : T(0);
        }
        EoT<N, T, 1> acc;
        acc.zero();
        const T sgn = s ? T(1) : T(-1);
        const T wgt = fam ? sc.area[2] : sc.area[1];
        auto flux = [&](T um, T up) {
          const T unm = sgn * lane_get(nl, um), unp = sgn * lane_get(nl, up);
          const T lam = fmax(fabs(unm), fabs(unp));
          return llf(um, up, unm, unp, lam, sc.lf, wgt);
        };
#pragma unroll
        for (int q1 = 0; q1 < (Q + 1) / 2; ++q1) {
          T ev[2], ov[2];   // even and odd parts at q1 and its mirror
#pragma unroll
          for (int sg = 0; sg < 2; ++sg) {
            ev[sg] = t.Sp[q1][0] * xe[sg][0];
            ov[sg] = t.Sm[q1][0] * xo[sg][0];
#pragma unroll
            for (int a = 1; a < NH; ++a) {
              ev[sg] = fmadd(t.Sp[q1][a], xe[sg][a], ev[sg]);
              ov[sg] = fmadd(t.Sm[q1][a], xo[sg][a], ov[sg]);
            }
            if constexpr (N % 2 == 1) ev[sg] = fmadd(t.Sc[q1], xm[sg], ev[sg]);
          }
          const T fq = flux(ev[0] + ov[0], ev[1] + ov[1]);
          if (q1 < QH) {
            const T fr = flux(ev[0] - ov[0], ev[1] - ov[1]);
            acc.pair(t.Tp[q1], t.Tm[q1], fq, fr);
          } else {
            acc.mid(t.Tc, fq);
          }
        }
#pragma unroll
        for (int c = 0; c < N; ++c) F[c * FP] = acc.out(c);
      }
    }

    // x pencils, items (j, q2, q3); after the face pencils, whose registers
    // would otherwise add to u_j
    const int j3 = tid / QQ, qq = tid - j3 * QQ;
    const bool own = tid < 3 * QQ;
    T* colb = lds + (own ? qq : 0);
    T* col = colb + (own ? j3 * COLS : 0);
    T* buf = colb + UBo;
    T U[Q];
    T F0 = 0, F1 = 0;   // x-face terms at the end nodes
    if constexpr (PERS) {   // defined on every path: nothing is carried over from the previous element
#pragma unroll
      for (int q = 0; q < Q; ++q) U[q] = T(0);
    }
    if (own) {
      T x[N];
      const T vL = col[0], vR = col[(N + 1) * SA];
#pragma unroll
      for (int c = 0; c < N; ++c) x[c] = col[(c + 1) * SA];
      const T unm0 = -colb[SA], unp0 = -colb[0], unm1 = colb[N * SA], unp1 = colb[(N + 1) * SA];
      SPLIT_TABLES(t);
      eo_interp<N, Q, T>(t, x, [&](int q, T v) { U[q] = v; });
      const T lam0 = fmax(fabs(unm0), fabs(unp0)), lam1 = fmax(fabs(unm1), fabs(unp1));
      F0 = llf(x[0], vL, unm0, unp0, lam0, sc.lf, sc.area[0]);
      F1 = llf(x[N - 1], vR, unm1, unp1, lam1, sc.lf, sc.area[0]);
    }

    // ---- passes over the flux direction f
    auto put_u = [&](int f) {
      if (own && j3 == f) {
#pragma unroll
        for (int q = 0; q < Q; ++q) buf[q * COLS] = U[q];
      }
    };
    // x back sweep of F_jf into the slots (own column only)
    auto xback = [&](auto fc) {
      constexpr int f = decltype(fc)::value;
      if (own) {
        SPLIT_TABLES(t);
        EoT<N, T, f == 0 ? -1 : 1> a;
        a.zero();
#pragma unroll
        for (int q = 0; q < QH; ++q) {
          const int rq = Q - 1 - q;
          const T xq = U[q] * buf[q * COLS], xr = U[rq] * buf[rq * COLS];
          if constexpr (f == 0) a.pair(t.Hp[q], t.Hm[q], xq, xr);
          else a.pair(t.Tp[q], t.Tm[q], xq, xr);
        }
        if constexpr (Q % 2 == 1) {
          const T xm = U[QH] * buf[QH * COLS];
          if constexpr (f == 0) a.mid(t.Hc, xm);
          else a.mid(t.Tc, xm);
        }
        const T s = sc.cell[f];
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T o = s * a.out(c);
          if constexpr (f == 0) {
            if (c == 0) o += F0;
            if (c == N - 1) o += F1;
          }
          col[c * SA] = o;
        }
      }
    };
    // back sweep of a pencil: a = S^T W or G^T W of the m values p[stride q]
    auto back = [&](auto& a, auto grad, const T* p, int stride) {
      SPLIT_TABLES(t);
      a.zero();
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        if constexpr (decltype(grad)::value) a.pair(t.Hp[q], t.Hm[q], p[stride * q], p[stride * (Q - 1 - q)]);
        else a.pair(t.Tp[q], t.Tm[q], p[stride * q], p[stride * (Q - 1 - q)]);
      }
      if constexpr (Q % 2 == 1) {
        if constexpr (decltype(grad)::value) a.mid(t.Hc, p[stride * QH]);
        else a.mid(t.Tc, p[stride * QH]);
      }
    };
    // y back sweep items (j, x node, q3) and z back sweep items (j, b, a)
    constexpr int nY = 3 * N * Q, nZ = 3 * N2;
    const int yq = tid % Q, yr = tid / Q, ya = yr % N, yj = yr / N;
    const bool ythr = tid < nY;
    T* ycol = lds + (ythr ? ya * SA + yj * COLS + yq : 0);
    const int zj = tid / N2, zab = tid - zj * N2, zb = zab / N, za = zab - zb * N;
    const bool zthr = tid < nZ;
    T* zcol = lds + (zthr ? za * SA + zj * COLS + Q * zb : 0);
    T Yk[N], Zk[N];
    if constexpr (PERS) {
#pragma unroll
      for (int c = 0; c < N; ++c) Yk[c] = Zk[c] = T(0);
    }

    bar();
    put_u(0);
    bar();
    xback(std::integral_constant<int, 0>{});
    bar();
    if (ythr) {
      EoT<N, T, 1> a;
      back(a, std::false_type{}, ycol, Q);
      const T* F = lds + FOo + yj * LAYER + ya * FP + yq;
#pragma unroll
      for (int b = 0; b < N; ++b) Yk[b] = a.out(b);
      Yk[0] += F[0];
      Yk[N - 1] += F[3 * LAYER];
    }
    {   // z-face terms: integrate in y, in place
      constexpr int nF = 6 * N, FI = wave_split(nY, nF, TH);
      for (int w = tid; w < FI + nF; w += TH) {
        if (w < FI) continue;
        const int v = w - FI, sj = v / N;   // sj = 3 s + j
        T* F = lds + FOo + FL + sj * LAYER + (v - sj * N) * FP;
        EoT<N, T, 1> a;
        back(a, std::false_type{}, F, 1);
#pragma unroll
        for (int b = 0; b < N; ++b) F[b] = a.out(b);
      }
    }
    put_u(1);
    bar();
    xback(std::integral_constant<int, 1>{});
    bar();
    if (ythr) {
      EoT<N, T, -1> a;
      back(a, std::true_type{}, ycol, Q);
#pragma unroll
      for (int b = 0; b < N; ++b) ycol[Q * b] = Yk[b] + a.out(b);
    }
    put_u(2);
    bar();
    if (zthr) {
      EoT<N, T, 1> a;
      back(a, std::false_type{}, zcol, 1);
      const T* F = lds + FOo + FL + zj * LAYER + za * FP + zb;
#pragma unroll
      for (int c = 0; c < N; ++c) Zk[c] = a.out(c);
      Zk[0] += F[0];
      Zk[N - 1] += F[3 * LAYER];
    }
    bar();
    xback(std::integral_constant<int, 2>{});
    if constexpr (PERS) issue(el + estep, el + estep < eend);   // u is done with: load the next element
    bar();
    if (ythr) {
      EoT<N, T, 1> a;
      back(a, std::false_type{}, ycol, Q);
#pragma unroll
      for (int b = 0; b < N; ++b) ycol[Q * b] = a.out(b);
    }
    bar();
    if (zthr) {
      EoT<N, T, -1> a;
      back(a, std::true_type{}, zcol, 1);
      T* g = r + zj * cs + (size_t)el * N3 + zab;
#pragma unroll
      for (int c = 0; c < N; ++c) g[N2 * c] = Zk[c] + a.out(c);
    }
    if constexpr (PERS) bar();   // the next element's P1 overwrites the slots read above
  }
}

// compute units of the current device, cached per device
static hipError_t cu_count(int* n) {
  static std::atomic<int> cache[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 64 && (*n = cache[dev].load(std::memory_order_relaxed)) > 0) return hipSuccess;
  e = hipDeviceGetAttribute(n, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess && *n < 1) e = hipErrorInvalidDevice;
  if (e == hipSuccess && dev < 64) cache[dev].store(*n, std::memory_order_relaxed);
  return e;
}

template <int N, int Q, typename T>
static hipError_t launch_split_nq(const ConvPlan& P, const void* u, void* r, hipStream_t s) {
  using Sh = SplitShape<N, Q, (int)sizeof(T)>;
  if (!conv_tables_match<N, Q>(P)) return hipErrorInvalidValue;
  ConvScal<T> sc;
  for (int d = 0; d < 3; ++d) {
    sc.cell[d] = (T)P.cell[d];
    sc.area[d] = (T)P.area[d];
  }
  sc.lf = (T)P.lf;
  const SplitTab<N, Q, T>* dt = nullptr;   // FP32 kernels use the compile-time tables
  if (sizeof(T) == 8) {
    hipError_t err;
    dt = plan_table<SplitTab<N, Q, T>>(
        P.tab.p[0], "convective_split", [&] { return make_split_tab<N, Q, T>(P.S.data(), P.G.data(), P.w.data()); }, &err);
    if (!dt) return err;
  }
  int grid = P.mesh.n_el;
  if (Sh::PERS) {
    int cus = 0;
    const hipError_t err = cu_count(&cus);
    if (err != hipSuccess) return err;
    grid = std::min(grid, cus);
  }
  hipLaunchKernelGGL((convective_split_kernel<N, Q, T, Sh::TH, Sh::PERS>), dim3(grid), dim3(Sh::TH), Sh::BYTES, s,
                     (const T*)u, (T*)r, P.mesh, dt, sc);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_split_t(const ConvPlan& P, const void* u, void* r, hipStream_t s) {
  switch (P.k) {
    case 4: return launch_split_nq<5, 7, T>(P, u, r, s);
    case 5: return launch_split_nq<6, 8, T>(P, u, r, s);
    case 6: return launch_split_nq<7, 10, T>(P, u, r, s);
    case 7: return launch_split_nq<8, 11, T>(P, u, r, s);
    case 8: return launch_split_nq<9, 13, T>(P, u, r, s);
    case 9: return launch_split_nq<10, 14, T>(P, u, r, s);
    case 10: return launch_split_nq<11, 16, T>(P, u, r, s);
    case 11: return launch_split_nq<12, 17, T>(P, u, r, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_convective_split(const ConvPlan& P, bool f32, const void* u, void* r, hipStream_t s) {
  return f32 ? launch_split_t<float>(P, u, r, s) : launch_split_t<double>(P, u, r, s);
}

}  // namespace dgmf
