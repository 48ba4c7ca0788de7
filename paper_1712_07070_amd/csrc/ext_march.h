// One z-march per padded patch group for the scheme words the default march
// (mhm_group.h) does not cover: PPM, CTU and dual energy, with any limiter,
// primitive or characteristic variables and any Riemann solver.
//
// Modes
//   kStep     MHM: face values, conservative Hancock half step, Riemann solves,
//             update (one launch per step)
//   kPredict  CTU, first pass: face values, each axis' own half step, first
//             Riemann solves at every face between two cells of [-1, 16]^3;
//             the differences of the first-solve fluxes across each cell go to
//             the workspace, [3 axes][NF][18^3] per group
//   kCorrect  CTU, second pass: the half-step states again, corrected with the
//             other two axes' flux differences, second solves, update
// CTU in one march would keep the states of two planes and the fluxes of both
// rounds per column: more than 256 registers per lane, or one wave per SIMD.
// The two passes recompute the predictor (PLM: a third of a pass) and move
// 15 (18) values per cell through HBM, against 75 for the chain of per-cell
// and per-face kernels.
//
// Mapping: 256 threads (4 waves, one per SIMD), a thread per interior (x, y)
// column; wave 0 also runs the 64 columns one cell outside the interior
// (x = -1, 16 and y = -1, 16) as a second pass through every phase, waves 1-3
// publish the columns further out (one per lane); wave 2 solves the 32 faces
// at x = 16 and y = 16 from states wave 0 leaves in LDS (kPredict: runs the 4
// corner columns, whose faces it solves itself as wave 0 does its own).  The
// march holds in registers what the z stencil needs; plane k goes through LDS
// for the x / y stencils:
//   publish   primitive plane k -> P                                | barrier
//   slopes    (PPM) limited x / y slopes of plane k -> D            | barrier
//   states    half-step states of plane k, x+ / y+ ones -> S; the z face
//             k - 1/2; update (kPredict: flux differences) of plane k - 1
//                                                                   | barrier
//   faces     x and y faces of plane k -> F
// PLM keeps the fluxes in an array of their own.  PPM reads them back in its
// extra phase, so the flux of a face takes the slot of the state on its low
// side, which only the thread that solves the face reads: 74 KB in FP64
// instead of 98, two workgroups per CU.
//
// A workgroup marches the planes of one z segment of its group, [z0, z1):
// with fewer groups than compute units a group's planes are shared by several
// workgroups (march_segments).  A segment of n planes runs n + 2 iterations,
// recomputing the states of one plane beyond each end and the face between
// two segments, which the upper one counts; the values are the same bits for
// any split.
//
// Bound by VALU issue and latency at two waves per SIMD.  256^3 FP64, ghost
// fill and step: PPM + hybrid + HLLC 6.70 -> 2.46 ms, CTU + PLM + Roe 10.0 ->
// 4.1 ms against the chain of per-cell kernels (scheme_ext.hip), whose passes
// over HBM bound it; 12 x 13 x 13 groups of noise, characteristic PPM + van
// Albada + HLLE 3.9 -> 1.26 ms; 210 groups FP32 with dual energy 0.210 -> 0.105.
// What cost most on the way: registers.  With the second-pass columns' stencils
// in registers wave 0 spilled 100 of them (PPM 3.2, CTU 5.3 ms: the spills
// went out to HBM); one wave per SIMD without spills took 3.5 and 4.8.
#pragma once

#include "march.h"
#include "mhm_group.h"

namespace gh {

__device__ __forceinline__ int ms_cell(int x, int y, int z) { return ((z + 1) * kMS + (y + 1)) * kMS + (x + 1); }

template <typename T, int NF, bool kPpm, int kMode>
struct XSmem {
  static constexpr int R = kPpm ? 2 : 1;  // reconstruction radius
  static constexpr int PW = kMS + 2 * R;  // primitive tile: x, y in [-1 - R, 16 + R]
  static constexpr int kPlane = kMS * kMS;
  static __device__ __forceinline__ int pi(int x, int y) { return (y + 1 + R) * PW + (x + 1 + R); }
  static __device__ __forceinline__ int si(int x, int y) { return (y + 1) * kMS + (x + 1); }
  static __device__ __forceinline__ int dxi(int x, int y) { return (y + 1) * 20 + (x + 2); }  // x in [-2, 17]
  static __device__ __forceinline__ int dyi(int x, int y) { return (y + 2) * kMS + (x + 1); }  // y in [-2, 17]
  T P[NF][PW * PW];                                        // primitive plane k
  T D[kPpm ? 2 : 1][kPpm ? NF : 1][kPpm ? 360 : 1];        // x and y slopes of plane k
  T S[2][NF][kPlane];                                      // x+ and y+ states of plane k
  T Fs[kPpm ? 1 : 2][kPpm ? 1 : NF][kPpm ? 1 : kPlane];    // fluxes, by the cell on the face's low side (PLM)
  T H[kMode == kPredict ? 1 : NF][32];                     // high-side states of the faces at x = 16, y = 16
  T C[kMode == kPredict ? 4 * NF : 1][68];                 // kPredict: Ux, Uy, Uz, Fz of the 64 + 4 second-pass columns
  T Z[kPpm ? 2 * NF : 1][68];                              // PPM: interface value and z slope of the second-pass columns
  // flux of the face of axis d whose low-side cell has state index i
  __device__ __forceinline__ T* flux(int d, int q) {
    if constexpr (kPpm) return S[d][q];
    else return Fs[d][q];
  }
};

// ------------------------------------------------------- reconstruction ----
template <int D, int NF, typename T>
__device__ __forceinline__ void march_slopes(const T Wm[NF], const T Wc[NF], const T Wp[NF], const Gas<T>& g,
                                             const ExtOpts& o, T s[NF]) {
  if (o.first_order) {
#pragma unroll
    for (int q = 0; q < NF; ++q) s[q] = T(0);
    return;
  }
  ext_slopes<D, false>(Wm, Wc, Wp, g, o, s);
  if constexpr (NF == 6) s[5] = passive_slope(Wm[5], Wc[5], Wp[5], g, o);
}

// Conserved form and flux of a face state; field 5: s = rho (s/rho), s u_n.
template <int D, int NF, typename T>
__device__ __forceinline__ void march_cons_flux(const T W[NF], const Gas<T>& g, T U[NF], T F[NF]) {
  ext_cons_flux<D>(W, g, U, F);
  if constexpr (NF == 6) {
    U[5] = W[0] * W[5];
    F[5] = U[5] * W[1 + D];
  }
}

template <int NF, typename T, class Src>
__device__ __forceinline__ void march_load(const Src& src, unsigned col, int z, T U[NF]) {
  const unsigned o = col + src.plane(z), fs = src.fstride();
#pragma unroll
  for (int q = 0; q < NF; ++q) U[q] = src.base[o + q * fs];
}

template <int NF, typename T>
__device__ __forceinline__ void march_prim(const T U[NF], const Gas<T>& g, T W[NF]) {
  cons_to_prim(U, g, W);
  if constexpr (NF == 6) W[5] = Fp<T>::div(U[5], U[0]);  // entropy per unit mass
}

// ------------------------------------------------------------- columns ----
// An interior column's z stencil between publishes: PLM W(k), W(k+1); PPM
// W(k+1), W(k+2), the z slope of plane k+1 and the interface value at k + 1/2
// (the high one of plane k and the low one of plane k+1).  zA, zB hold what
// plane k's z face values are made of: PLM its slope (zA); PPM the interface
// values at k -+ 1/2.  W(k) itself is read back from P.
template <typename T, int NF, bool kPpm>
struct XCol {
  int cx, cy;
  unsigned col;
  T W0[NF], W1[NF];    // at the start of iteration k: PLM W(k-1), W(k); PPM W(k), W(k+1)
  T s0[kPpm ? NF : 1]; // PPM: z slope of plane k
  T zA[NF];
  T zB[kPpm ? NF : 1];
  T Un[NF];            // conserved plane k+1 (PLM) or k+2 (PPM), in flight
};

template <typename T, int NF, bool kPpm>
__device__ __forceinline__ void xcol_load(XCol<T, NF, kPpm>& c, const PaddedSource<T>& src, int k, int z1) {
  constexpr int a = kPpm ? 2 : 1;
  march_load<NF>(src, c.col, k <= z1 ? k + a : z1 + a, c.Un);  // clamped, so unconditional
}

// PPM: z slope of plane z0-1 and interface value at z0 - 3/2, from the
// primitive planes z0-3 .. z0.
template <int NF, typename T>
__device__ __forceinline__ void ppm_z_start(const PaddedSource<T>& src, unsigned col, int z0, const Gas<T>& gas,
                                            const ExtOpts& o, T W0[NF], T W1[NF], T s0[NF], T I[NF]) {
  T U[NF], a[NF], b[NF], s[NF];
  march_load<NF>(src, col, z0 - 3, U);
  march_prim<NF>(U, gas, a);
  march_load<NF>(src, col, z0 - 2, U);
  march_prim<NF>(U, gas, b);
  march_load<NF>(src, col, z0 - 1, U);
  march_prim<NF>(U, gas, W0);
  march_load<NF>(src, col, z0, U);
  march_prim<NF>(U, gas, W1);
  march_slopes<2, NF>(a, b, W0, gas, o, s);
  march_slopes<2, NF>(b, W0, W1, gas, o, s0);
#pragma unroll
  for (int q = 0; q < NF; ++q) I[q] = ppm_interface(b[q], W0[q], s[q], s0[q]);
}

template <typename T, int NF, bool kPpm>
__device__ __forceinline__ void xcol_init(XCol<T, NF, kPpm>& c, const PaddedSource<T>& src, int cx, int cy, int z0,
                                          int z1, const Gas<T>& gas, const ExtOpts& o) {
  c.cx = cx;
  c.cy = cy;
  c.col = src.col(cx, cy);
  if constexpr (kPpm) {
    ppm_z_start<NF>(src, c.col, z0, gas, o, c.W0, c.W1, c.s0, c.zB);
  } else {
    T U[NF];
    march_load<NF>(src, c.col, z0 - 2, U);
    march_prim<NF>(U, gas, c.W0);
    march_load<NF>(src, c.col, z0 - 1, U);
    march_prim<NF>(U, gas, c.W1);
  }
  xcol_load(c, src, z0 - 1, z1);
}

// Publish plane k and take in the plane that arrived.
template <typename T, int NF, bool kPpm, class Sm>
__device__ __forceinline__ void xcol_publish(XCol<T, NF, kPpm>& c, const Gas<T>& gas, const ExtOpts& o, Sm& sm) {
#pragma unroll
  for (int q = 0; q < NF; ++q) sm.P[q][sm.pi(c.cx, c.cy)] = kPpm ? c.W0[q] : c.W1[q];
  T W2[NF], s1[NF];
  march_prim<NF>(c.Un, gas, W2);
  march_slopes<2, NF>(c.W0, c.W1, W2, gas, o, s1);
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    if constexpr (kPpm) {
      c.zA[q] = c.zB[q];
      c.zB[q] = ppm_interface(c.W0[q], c.W1[q], c.s0[q], s1[q]);
      c.s0[q] = s1[q];
    } else {
      c.zA[q] = s1[q];
    }
    c.W0[q] = c.W1[q];
    c.W1[q] = W2[q];
  }
}

// A second-pass column keeps no registers from one iteration to the next but
// the loads in flight (three conserved planes, re-read from the caches): with
// its stencil in registers the wave that runs it beside its interior columns
// would spill.  PPM's slope and interface value wait in LDS (Sm::Z).
template <typename T, int NF, bool kPpm>
struct XCol2 {
  int cx, cy, slot;
  unsigned col;
  T U[3][NF];  // conserved planes k-1, k, k+1 (PLM) or k, k+1, k+2 (PPM), in flight
  T zA[NF];    // PLM: z slope of plane k; PPM: interface value at k + 1/2
};

template <typename T, int NF, bool kPpm>
__device__ __forceinline__ void xcol2_load(XCol2<T, NF, kPpm>& c, const PaddedSource<T>& src, int k, int z1) {
  const int z = (k <= z1 ? k : z1) - (kPpm ? 0 : 1);
#pragma unroll
  for (int j = 0; j < 3; ++j) march_load<NF>(src, c.col, z + j, c.U[j]);
}

template <typename T, int NF, bool kPpm, class Sm>
__device__ __forceinline__ void xcol2_init(XCol2<T, NF, kPpm>& c, const PaddedSource<T>& src, int cx, int cy, int slot,
                                           int z0, int z1, const Gas<T>& gas, const ExtOpts& o, Sm& sm) {
  c.cx = cx;
  c.cy = cy;
  c.slot = slot;
  c.col = src.col(cx, cy);
  if constexpr (kPpm) {
    T W0[NF], W1[NF], s0[NF], I[NF];
    ppm_z_start<NF>(src, c.col, z0, gas, o, W0, W1, s0, I);
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      sm.Z[q][slot] = I[q];
      sm.Z[NF + q][slot] = s0[q];
    }
  }
  xcol2_load(c, src, z0 - 1, z1);
}

template <typename T, int NF, bool kPpm, class Sm>
__device__ __forceinline__ void xcol2_publish(XCol2<T, NF, kPpm>& c, const Gas<T>& gas, const ExtOpts& o, Sm& sm) {
  T W[3][NF], s1[NF];
#pragma unroll
  for (int j = 0; j < 3; ++j) march_prim<NF>(c.U[j], gas, W[j]);
#pragma unroll
  for (int q = 0; q < NF; ++q) sm.P[q][sm.pi(c.cx, c.cy)] = W[kPpm ? 0 : 1][q];
  march_slopes<2, NF>(W[0], W[1], W[2], gas, o, s1);
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    if constexpr (kPpm) {
      c.zA[q] = ppm_interface(W[0][q], W[1][q], sm.Z[NF + q][c.slot], s1[q]);
      sm.Z[NF + q][c.slot] = s1[q];
    } else {
      c.zA[q] = s1[q];
    }
  }
}

// PPM: x and y slopes of plane k at (x, y).
template <int NF, typename T, class Sm>
__device__ __forceinline__ void xslope_x(int x, int y, const Gas<T>& gas, const ExtOpts& o, Sm& sm) {
  T a[NF], b[NF], c[NF], s[NF];
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    a[q] = sm.P[q][sm.pi(x - 1, y)];
    b[q] = sm.P[q][sm.pi(x, y)];
    c[q] = sm.P[q][sm.pi(x + 1, y)];
  }
  march_slopes<0, NF>(a, b, c, gas, o, s);
#pragma unroll
  for (int q = 0; q < NF; ++q) sm.D[0][q][sm.dxi(x, y)] = s[q];
}
template <int NF, typename T, class Sm>
__device__ __forceinline__ void xslope_y(int x, int y, const Gas<T>& gas, const ExtOpts& o, Sm& sm) {
  T a[NF], b[NF], c[NF], s[NF];
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    a[q] = sm.P[q][sm.pi(x, y - 1)];
    b[q] = sm.P[q][sm.pi(x, y)];
    c[q] = sm.P[q][sm.pi(x, y + 1)];
  }
  march_slopes<1, NF>(a, b, c, gas, o, s);
#pragma unroll
  for (int q = 0; q < NF; ++q) sm.D[1][q][sm.dyi(x, y)] = s[q];
}

// Half-step states of the cell (cx, cy) at plane k: the x+ / y+ ones to S, the
// others to Ux, Uy (low faces) and zl, zh.  zA, zB: XCol's.  corr(d, q):
// kCorrect's correction of axis d.  One axis at a time, and the x+ / y+ states
// wait in their own S slots (not in registers) for the sum of the three axes'
// flux differences that completes MHM's half step.
template <int kMode, int NF, bool kPpm, typename T, class Sm, class Corr>
__device__ __forceinline__ void half_step(int cx, int cy, const T zA[NF], const T zB[NF], const Gas<T>& gas,
                                          const ExtOpts& o, Sm& sm, T Ux[NF], T Uy[NF], T zl[NF], T zh[NF],
                                          const Corr& corr) {
  const int i0 = sm.si(cx, cy);
  T Wc[NF], sum[NF];
#pragma unroll
  for (int q = 0; q < NF; ++q) Wc[q] = sm.P[q][sm.pi(cx, cy)];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int xm = d == 0 ? cx - 1 : cx, xp = d == 0 ? cx + 1 : cx;
    const int ym = d == 1 ? cy - 1 : cy, yp = d == 1 ? cy + 1 : cy;
    T lo[NF], hi[NF];
    if constexpr (kPpm) {
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        if (d == 2) {
          lo[q] = zA[q];
          hi[q] = zB[q];
        } else {
          const T* S = sm.D[d == 0 ? 0 : 1][q];
          const T sm_ = S[d == 0 ? sm.dxi(xm, cy) : sm.dyi(cx, ym)];
          const T s0_ = S[d == 0 ? sm.dxi(cx, cy) : sm.dyi(cx, cy)];
          const T sp_ = S[d == 0 ? sm.dxi(xp, cy) : sm.dyi(cx, yp)];
          lo[q] = ppm_interface(sm.P[q][sm.pi(xm, ym)], Wc[q], sm_, s0_);
          hi[q] = ppm_interface(Wc[q], sm.P[q][sm.pi(xp, yp)], s0_, sp_);
        }
        if (o.first_order) lo[q] = hi[q] = Wc[q];
        else ppm_monotone(Wc[q], lo[q], hi[q]);
      }
    } else {
      T s[NF];
      if (d == 2) {
#pragma unroll
        for (int q = 0; q < NF; ++q) s[q] = zA[q];
      } else {
        T Wa[NF], Wb[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          Wa[q] = sm.P[q][sm.pi(xm, ym)];
          Wb[q] = sm.P[q][sm.pi(xp, yp)];
        }
        if (d == 0) march_slopes<0, NF>(Wa, Wc, Wb, gas, o, s);
        else march_slopes<1, NF>(Wa, Wc, Wb, gas, o, s);
      }
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        lo[q] = Wc[q] - T(0.5) * s[q];
        hi[q] = Wc[q] + T(0.5) * s[q];
      }
    }
    T* Ul = d == 0 ? Ux : d == 1 ? Uy : zl;
    T Uh[NF], Fl[NF], Fh[NF];
    if (d == 0) {
      march_cons_flux<0, NF>(lo, gas, Ul, Fl);
      march_cons_flux<0, NF>(hi, gas, Uh, Fh);
    } else if (d == 1) {
      march_cons_flux<1, NF>(lo, gas, Ul, Fl);
      march_cons_flux<1, NF>(hi, gas, Uh, Fh);
    } else {
      march_cons_flux<2, NF>(lo, gas, Ul, Fl);
      march_cons_flux<2, NF>(hi, gas, Uh, Fh);
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      const T dF = Fl[q] - Fh[q];
      if constexpr (kMode == kStep) {
        sum[q] = d == 0 ? dF : sum[q] + dF;
      } else {
        const T dU = gas.half_dtdx * dF;  // CTU: the axis' own flux difference
        Ul[q] = Ul[q] + dU;
        Uh[q] = Uh[q] + dU;
        if constexpr (kMode == kCorrect) {
          const T cq = corr(d, q);
          Ul[q] = Ul[q] - gas.half_dtdx * cq;
          Uh[q] = Uh[q] - gas.half_dtdx * cq;
        }
      }
      if (d < 2) sm.S[d][q][i0] = Uh[q];
      else zh[q] = Uh[q];
    }
  }
  if constexpr (kMode == kStep) {
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      const T dU = gas.half_dtdx * sum[q];
      sm.S[0][q][i0] = sm.S[0][q][i0] + dU;
      sm.S[1][q][i0] = sm.S[1][q][i0] + dU;
      Ux[q] = Ux[q] + dU;
      Uy[q] = Uy[q] + dU;
      zl[q] = zl[q] + dU;
      zh[q] = zh[q] + dU;
    }
  }
}

__device__ __forceinline__ double march_pow(double x, double e) { return ::pow(x, e); }
__device__ __forceinline__ float march_pow(float x, float e) { return ::powf(x, e); }

enum MarchRole { kMarchHalo = 0, kMarchPlain = 1, kMarchLast = 2 };

// The march of one wave.  Every role passes the same barriers.
template <typename T, int NF, bool kPpm, int kMode, int kRole, class Sm>
__device__ __forceinline__ int xmarch(const MarchArgs<T>& A, const PaddedSource<T>& src, const Gas<T>& gas,
                                      const ExtOpts& o, int64_t g, int z0, int z1, Sm& sm, int tid) {
  constexpr bool kPre = kMode == kPredict;
  // the second-pass columns: wave 0's 64, in kPredict also wave 2's 4 corners
  constexpr bool kSecond = kRole == kMarchHalo || (kPre && kRole == kMarchLast);
  const int lane = tid & 63, wave = tid >> 6;
  T* out = A.U_out + g * NF * 4096;
  T* dFg = A.dF + g * 3 * NF * int64_t(kMS3);
  T* ff = (NF == 5 && !kPre && A.face_flux != nullptr) ? A.face_flux + g * 9 * 5 * 256 : nullptr;

  XCol<T, NF, kPpm> ci;
  XCol2<T, NF, kPpm> cs;
  xcol_init(ci, src, tid & 15, tid >> 4, z0, z1, gas, o);
  const bool second = kRole == kMarchHalo || (kSecond && lane < 4);
  if (kSecond) {
    if (kRole == kMarchHalo) {
      const int side = lane >> 4, kk = lane & 15;
      xcol2_init(cs, src, side == 0 ? -1 : side == 1 ? 16 : kk, side == 2 ? -1 : side == 3 ? 16 : kk, lane, z0, z1,
                 gas, o, sm);
    } else {
      xcol2_init(cs, src, (lane & 1) ? 16 : -1, (lane & 2) ? 16 : -1, 64 + (lane & 3), z0, z1, gas, o, sm);
    }
  }

  // columns further out, one per lane of waves 1-3 (only published):
  //   wave 1: x = -2, 17 (36); wave 3: y = -2, 17 (36); wave 2: the 4
  //   corners (kPredict runs them as columns); PPM also x, y = -3, 18 (72:
  //   28 on waves 1 and 3 each, 16 on wave 2)
  int ex = 0, ey = 0;
  bool has_extra = false, slope_x = false, slope_y = false;
  if (kRole != kMarchHalo) {
    const int a = lane % kMS - 1;
    int deep = -1;
    if (kRole == kMarchLast) {
      if (lane < 4) {
        ex = (lane & 1) ? 16 : -1;
        ey = (lane & 2) ? 16 : -1;
        has_extra = !kPre;
        slope_x = slope_y = true;
      } else if (kPpm && lane < 20) {
        deep = 56 + lane - 4;
      }
    } else if (lane < 2 * kMS) {
      const int b = lane < kMS ? -2 : 17;
      ex = wave == 1 ? b : a;
      ey = wave == 1 ? a : b;
      has_extra = true;
      slope_x = wave == 1;
      slope_y = wave == 3;
    } else if (kPpm) {
      deep = (wave == 1 ? 0 : 28) + lane - 2 * kMS;
    }
    if (kPpm && deep >= 0) {
      const int j = deep % 36, c = j % kMS - 1, b = j < kMS ? -3 : 18;
      ex = deep < 36 ? b : c;
      ey = deep < 36 ? c : b;
      has_extra = true;
    }
  }
  unsigned col_ex = 0;
  T Ue[NF];
  if (kRole != kMarchHalo) {
    col_ex = src.col(ex, ey);
    march_load<NF>(src, col_ex, z0 - 1, Ue);
  }

  // interior column: z+ state of plane k-1, z flux at the low face of plane
  // k-1, x / y flux differences of plane k-1
  T Uz[NF], Fz0[NF], acc[NF];
  int bad = 0;
  const int klo = (kPre && z0 == 0) ? -1 : z0, khi = (kPre && z1 == 16) ? 16 : z1 - 1;  // planes of x / y faces

  // kPredict: differences of the x / y fluxes of plane j across the column's
  // cell, where both faces exist
  auto put_dxy = [&](int x, int y, int j) {
    const int i0 = sm.si(x, y), c = ms_cell(x, y, j);
    if (x >= 0 && x <= 15) {
#pragma unroll
      for (int q = 0; q < NF; ++q) dFg[(0 * NF + q) * int64_t(kMS3) + c] = sm.flux(0, q)[i0] - sm.flux(0, q)[i0 - 1];
    }
    if (y >= 0 && y <= 15) {
#pragma unroll
      for (int q = 0; q < NF; ++q) dFg[(1 * NF + q) * int64_t(kMS3) + c] = sm.flux(1, q)[i0] - sm.flux(1, q)[i0 - kMS];
    }
  };

#pragma unroll 1
  for (int k = z0 - 1; k <= z1; ++k) {
    // ---- publish plane k
    xcol_publish(ci, gas, o, sm);
    if (kSecond && second) xcol2_publish(cs, gas, o, sm);
    if (kRole != kMarchHalo && has_extra) {
      T We[NF];
      march_prim<NF>(Ue, gas, We);
#pragma unroll
      for (int q = 0; q < NF; ++q) sm.P[q][sm.pi(ex, ey)] = We[q];
    }
    __syncthreads();

    // ---- fluxes of plane k-1 (before S, and with it PPM's flux slots, is rewritten)
    auto take_fluxes = [&]() {
      if constexpr (kPre) {
        if (k - 1 >= klo) {
          put_dxy(ci.cx, ci.cy, k - 1);
          if (kSecond && second) put_dxy(cs.cx, cs.cy, k - 1);
        }
      } else if (k > z0) {
        const int i0 = sm.si(ci.cx, ci.cy);
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          acc[q] = sm.flux(0, q)[i0] - sm.flux(0, q)[i0 - 1];
          acc[q] = acc[q] + (sm.flux(1, q)[i0] - sm.flux(1, q)[i0 - kMS]);
        }
      }
    };
    take_fluxes();
    if constexpr (kPpm) {
      xslope_x<NF>(ci.cx, ci.cy, gas, o, sm);
      xslope_y<NF>(ci.cx, ci.cy, gas, o, sm);
      if (kSecond && second) {
        xslope_x<NF>(cs.cx, cs.cy, gas, o, sm);
        xslope_y<NF>(cs.cx, cs.cy, gas, o, sm);
      }
      if (kRole == kMarchPlain) {
        if (slope_x) xslope_x<NF>(ex, ey, gas, o, sm);
        if (slope_y) xslope_y<NF>(ex, ey, gas, o, sm);
      }
      if (kRole == kMarchLast && !kPre && slope_x) {
        xslope_x<NF>(ex, ey, gas, o, sm);
        xslope_y<NF>(ex, ey, gas, o, sm);
      }
      __syncthreads();
    }

    // ---- states of plane k: second-pass columns first (nothing of the
    // interior column's is live yet but its z stencil)
    if (kSecond && second && (kPre || (k >= z0 && k < z1))) {
      // kCorrect: only the states on the face the column shares with the
      // interior are used; theirs is the transverse and the z difference
      const int ta = cs.cx < 0 || cs.cx > 15 ? 1 : 0, c = ms_cell(cs.cx, cs.cy, k);
      T hx[NF], hy[NF], zl[NF], zh[NF], zA[NF];
#pragma unroll
      for (int q = 0; q < NF; ++q) zA[q] = kPpm ? sm.Z[q][cs.slot] : cs.zA[q];
      half_step<kMode, NF, kPpm>(cs.cx, cs.cy, zA, cs.zA, gas, o, sm, hx, hy, zl, zh, [&](int d, int q) {
        return d == 2 ? T(0) : dFg[(ta * NF + q) * int64_t(kMS3) + c] + dFg[(2 * NF + q) * int64_t(kMS3) + c];
      });
      if constexpr (kPre) {
        if (kRole == kMarchHalo && k >= z0) {  // no z differences are needed at the corners
          T L[NF], Fz1[NF];
#pragma unroll
          for (int q = 0; q < NF; ++q) L[q] = sm.C[2 * NF + q][cs.slot];
          riemann_nf<2, NF>(L, zl, gas, o, Fz1);
          const int cz = ms_cell(cs.cx, cs.cy, k - 1);
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            if (k > z0) dFg[(2 * NF + q) * int64_t(kMS3) + cz] = Fz1[q] - sm.C[3 * NF + q][cs.slot];
            sm.C[3 * NF + q][cs.slot] = Fz1[q];
          }
        }
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          sm.C[q][cs.slot] = hx[q];
          sm.C[NF + q][cs.slot] = hy[q];
          sm.C[2 * NF + q][cs.slot] = zh[q];
        }
      } else if (cs.cx == 16 || cs.cy == 16) {
        const int slot = cs.cx == 16 ? cs.cy : 16 + cs.cx;
#pragma unroll
        for (int q = 0; q < NF; ++q) sm.H[q][slot] = cs.cx == 16 ? hx[q] : hy[q];
      }
    }
    if constexpr (kPpm) {
      if (kSecond && second) {
#pragma unroll
        for (int q = 0; q < NF; ++q) sm.Z[q][cs.slot] = cs.zA[q];
      }
    }
    T Ux[NF], Uy[NF], zl[NF], zh[NF];
    half_step<kMode, NF, kPpm>(ci.cx, ci.cy, ci.zA, ci.zB, gas, o, sm, Ux, Uy, zl, zh, [&](int d, int q) {
      // the other two axes' differences at the cell; z differences exist for
      // planes 0..15 (planes -1 and 16 use their z states only)
      const int c = ms_cell(ci.cx, ci.cy, d == 2 ? k : (k < 0 ? 0 : (k > 15 ? 15 : k)));
      const int a = d == 0 ? 1 : 0, b = d == 2 ? 1 : 2;
      return dFg[(a * NF + q) * int64_t(kMS3) + c] + dFg[(b * NF + q) * int64_t(kMS3) + c];
    });
    __syncthreads();

    // ---- x and y faces of plane k
    if (k >= klo && k <= khi) {
      const int i0 = sm.si(ci.cx, ci.cy);
      T Lx[NF], Ly[NF], Fx[NF], Fy[NF];
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        Lx[q] = sm.S[0][q][i0 - 1];
        Ly[q] = sm.S[1][q][i0 - kMS];
      }
      // one after the other: solved together (hllc_flux2) they spill in FP64
      // with PPM (256^3 step 2.62 -> 3.34 ms)
      const int b = int(riemann_nf<0, NF>(Lx, Ux, gas, o, Fx)) + int(riemann_nf<1, NF>(Ly, Uy, gas, o, Fy));
      if (!kPre) bad += b;
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        sm.flux(0, q)[i0 - 1] = Fx[q];
        sm.flux(1, q)[i0 - kMS] = Fy[q];
      }
      if (!kPre && ff != nullptr) {
        if ((ci.cx & 7) == 0) {
          T* of = ff + (ci.cx >> 3) * 5 * 256 + k * 16 + ci.cy;
#pragma unroll
          for (int q = 0; q < 5; ++q) of[q * 256] = Fx[q];
        }
        if ((ci.cy & 7) == 0) {
          T* of = ff + (3 + (ci.cy >> 3)) * 5 * 256 + ci.cx * 16 + k;
#pragma unroll
          for (int q = 0; q < 5; ++q) of[q * 256] = Fy[q];
        }
      }
      if constexpr (kPre) {
        if (kSecond && second) {
          const int j0 = sm.si(cs.cx, cs.cy);
          T L[NF], Rr[NF], F[NF];
          if (cs.cx >= 0) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
              L[q] = sm.S[0][q][j0 - 1];
              Rr[q] = sm.C[q][cs.slot];
            }
            riemann_nf<0, NF>(L, Rr, gas, o, F);
#pragma unroll
            for (int q = 0; q < NF; ++q) sm.flux(0, q)[j0 - 1] = F[q];
          }
          if (cs.cy >= 0) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
              L[q] = sm.S[1][q][j0 - kMS];
              Rr[q] = sm.C[NF + q][cs.slot];
            }
            riemann_nf<1, NF>(L, Rr, gas, o, F);
#pragma unroll
            for (int q = 0; q < NF; ++q) sm.flux(1, q)[j0 - kMS] = F[q];
          }
        }
      } else if (kRole == kMarchLast && lane < 32) {
        // the faces at x = 16 (lanes 0..15, y = lane) and y = 16 (x = lane -
        // 16) in one pass, the y faces rotated into the x-normal frame
        const bool yf = lane >= 16;
        const int i = lane & 15, low = yf ? sm.si(i, 15) : sm.si(15, i);
        T L[NF], Rr[NF], Lr[NF], Rn[NF], F[NF], Fo[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          L[q] = yf ? sm.S[1][q][low] : sm.S[0][q][low];
          Rr[q] = sm.H[q][lane];
        }
        auto rot = [&](const T a[NF], T r[NF]) {
          r[0] = a[0];
          r[1] = yf ? a[2] : a[1];
          r[2] = yf ? a[3] : a[2];
          r[3] = yf ? a[1] : a[3];
          r[4] = a[4];
          if constexpr (NF == 6) r[5] = a[5];
        };
        rot(L, Lr);
        rot(Rr, Rn);
        bad += riemann_nf<0, NF>(Lr, Rn, gas, o, F) ? 1 : 0;
        Fo[0] = F[0];
        Fo[1] = yf ? F[3] : F[1];
        Fo[2] = yf ? F[1] : F[2];
        Fo[3] = yf ? F[2] : F[3];
        Fo[4] = F[4];
        if constexpr (NF == 6) Fo[5] = F[5];
#pragma unroll
        for (int q = 0; q < NF; ++q) (yf ? sm.flux(1, q) : sm.flux(0, q))[low] = Fo[q];
        if (ff != nullptr) {
          T* of = ff + (yf ? 5 * 5 * 256 + i * 16 + k : 2 * 5 * 256 + k * 16 + i);
#pragma unroll
          for (int q = 0; q < 5; ++q) of[q * 256] = Fo[q];
        }
      }
    }

    // ---- z face k - 1/2; plane k-1 completed
    if (k >= z0) {
      T Uold[NF], Fz1[NF];
      if (!kPre && k > z0) march_load<NF>(src, ci.col, k - 1, Uold);
      const int b = riemann_nf<2, NF>(Uz, zl, gas, o, Fz1) ? 1 : 0;
      const bool own = k < z1 || z1 == 16;  // the face between two segments belongs to the upper one
      if (!kPre && own) bad += b;
      if (!kPre && own && ff != nullptr && (k & 7) == 0) {
        T* of = ff + (6 + (k >> 3)) * 5 * 256 + ci.cy * 16 + ci.cx;
#pragma unroll
        for (int q = 0; q < 5; ++q) of[q * 256] = Fz1[q];
      }
      if (k > z0) {
        if constexpr (kPre) {
          const int c = ms_cell(ci.cx, ci.cy, k - 1);
#pragma unroll
          for (int q = 0; q < NF; ++q) dFg[(2 * NF + q) * int64_t(kMS3) + c] = Fz1[q] - Fz0[q];
        } else {
          T Un[NF];
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            const T a = acc[q] + (Fz1[q] - Fz0[q]);
            Un[q] = Uold[q] - gas.dtdx * a;
          }
          if constexpr (NF == 6) {
            // dual energy: E from the entropy where E_th < xi E_kin, else
            // the entropy from E
            const T ekin = T(0.5) * (Un[1] * Un[1] + Un[2] * Un[2] + Un[3] * Un[3]) * Fp<T>::rcp(Un[0]);
            const T eth = Un[4] - ekin;
            const T rg = march_pow(Un[0], gas.gm1);
            if (eth < A.xi * ekin) Un[4] = Un[5] * rg * gas.inv_gm1 + ekin;
            else Un[5] = Fp<T>::div(gas.gm1 * eth, rg);
          }
#pragma unroll
          for (int q = 0; q < NF; ++q) out[q * 4096 + ((k - 1) * 16 + ci.cy) * 16 + ci.cx] = Un[q];
          bad += unphysical(Un, gas) ? 1 : 0;
        }
      }
#pragma unroll
      for (int q = 0; q < NF; ++q) Fz0[q] = Fz1[q];
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) Uz[q] = zh[q];
    // the next iteration's planes: issued here, where the fewest registers
    // are live, rather than an iteration ahead (256^3 FP64 PPM 2.62 -> 2.45,
    // CTU 4.24 -> 3.99 ms; the loads hit the caches)
    asm volatile("" ::: "memory");
    xcol_load(ci, src, k + 1, z1);
    if (kSecond) xcol2_load(cs, src, k + 1, z1);
    if (kRole != kMarchHalo) march_load<NF>(src, col_ex, k < z1 ? k + 1 : z1, Ue);
  }
  if constexpr (kPre) {
    if (z1 == 16) {  // uniform: the x / y differences of the last plane
      __syncthreads();
      put_dxy(ci.cx, ci.cy, 16);
      if (kSecond && second) put_dxy(cs.cx, cs.cy, 16);
    }
  }
  return bad;
}

// kChr: characteristic variables; kRoe 1: Roe, 0: HLLC or HLLE (run time).
template <typename T, int NF, bool kPpm, int kMode, int kChr, int kRoe>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(sizeof(XSmem<T, NF, kPpm, kMode>) > 81920 ? 1 : 2))) void march_kernel(MarchArgs<T> A) {
  __shared__ XSmem<T, NF, kPpm, kMode> sm;
  Gas<T> gas = A.gas;
  set_dt(gas, A.dt_dev, A.dx);
  ExtOpts o = A.o;
  o.ctu = kMode != kStep;
  o.ppm = kPpm;
  o.chr = kChr;
  o.solver = kRoe ? 1 : (A.o.solver == 2 ? 2 : 0);
  const int64_t g = blockIdx.x / unsigned(A.segs);
  const int n = 16 / A.segs, z0 = int(blockIdx.x % unsigned(A.segs)) * n, z1 = z0 + n;
  const int P = 16 + 2 * A.gh;
  PaddedSource<T> src{A.U_pad + g * NF * int64_t(P) * P * P, P, A.gh};
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bad;
  if (wave == 0) bad = xmarch<T, NF, kPpm, kMode, kMarchHalo>(A, src, gas, o, g, z0, z1, sm, tid);
  else if (wave == 2) bad = xmarch<T, NF, kPpm, kMode, kMarchLast>(A, src, gas, o, g, z0, z1, sm, tid);
  else bad = xmarch<T, NF, kPpm, kMode, kMarchPlain>(A, src, gas, o, g, z0, z1, sm, tid);
  if (kMode != kPredict && A.n_bad != nullptr && bad != 0) atomicAdd(A.n_bad, bad);
}

// Workgroups of a kernel that fit on a compute unit.
inline int march_slots(const void* kernel) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kThreads, 0) != hipSuccess || n < 1) n = 1;
  return n;
}

template <typename T, int NF, bool kPpm, int kMode, int kChr, int kRoe>
void launch_march_copy(MarchArgs<T>& A, int64_t n, hipStream_t stream) {
  static const int slots = march_slots(reinterpret_cast<const void*>(march_kernel<T, NF, kPpm, kMode, kChr, kRoe>));
  A.segs = march_segments(n, slots, sizeof(T) == 8 ? 0.36 : 0.15);
  hipLaunchKernelGGL((march_kernel<T, NF, kPpm, kMode, kChr, kRoe>), dim3(unsigned(n * A.segs)), dim3(kThreads), 0,
                     stream, A);
}

// Launch one mode of the march over G groups (in launches of at most 2^26
// groups).
template <typename T, int NF, bool kPpm, int kMode>
hipError_t launch_march_mode(const MarchArgs<T>& args, int64_t G, hipStream_t stream) {
  const int64_t chunk = int64_t(1) << 26;
  const int64_t P = 16 + 2 * args.gh;
  for (int64_t g0 = 0; g0 < G; g0 += chunk) {
    const int64_t n = G - g0 < chunk ? G - g0 : chunk;
    MarchArgs<T> A = args;
    A.U_pad += g0 * NF * P * P * P;
    A.U_out += g0 * NF * 4096;
    if (A.face_flux != nullptr) A.face_flux += g0 * 9 * 5 * 256;
    if (A.dF != nullptr) A.dF += g0 * 3 * NF * int64_t(kMS3);
    const bool roe = A.o.solver == 1;
    if (A.o.chr) {
      if (roe) launch_march_copy<T, NF, kPpm, kMode, 1, 1>(A, n, stream);
      else launch_march_copy<T, NF, kPpm, kMode, 1, 0>(A, n, stream);
    } else {
      if (roe) launch_march_copy<T, NF, kPpm, kMode, 0, 1>(A, n, stream);
      else launch_march_copy<T, NF, kPpm, kMode, 0, 0>(A, n, stream);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gh
