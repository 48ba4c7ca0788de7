// Per-group device code of the MHM step shared by the level kernels
// (mhm_fwd.hip) and the batched persistent kernel (mhm_batched.hip): input
// sources, the LDS layout, and the z-marching routine that advances one
// 16^3 patch group with one 256-thread workgroup (the mapping of threads to
// columns and roles is described at "one patch group" below).
#pragma once

#include <type_traits>

#include "ext_device.h"
#include "hydro_device.h"
#include "kernels.h"

namespace gh {

constexpr int kThreads = 256;
constexpr int kPW = 20;  // primitive plane tile: x, y in [-2, 17]
constexpr int kSW = 18;  // state tile: x, y in [-1, 16]

__device__ __forceinline__ int pidx(int x, int y) { return (y + 2) * kPW + (x + 2); }
__device__ __forceinline__ int sidx(int x, int y) { return (y + 1) * kSW + (x + 1); }
__device__ __forceinline__ int fxidx(int i, int j) { return j * 17 + i; }  // x-face i: between i-1 and i
__device__ __forceinline__ int fyidx(int i, int j) { return j * 16 + i; }  // y-face j: between j-1 and j

// ------------------------------------------------------------- sources ----
// A source maps group-relative cell coordinates to element offsets:
// offset(f, x, y, z) = col(x, y) + plane(z) + f * fstride, in the source's
// offset type Off.  A 32-bit unsigned offset lets every load take the
// scalar-base + 32-bit-vector-offset address form (no 64-bit address adds in
// the march, fewer registers: measured 1-5% per step); sources that can hold
// 2^32 elements or more use 64-bit offsets.

template <typename T>
struct PaddedSource {
  using Off = unsigned int;  // one group's padded block: 5 P^3 elements
  const T* base;  // this group's padded block
  int P, gh;
  __device__ Off col(int x, int y) const { return Off(y + gh) * P + (x + gh); }
  __device__ Off plane(int z) const { return Off(z + gh) * P * P; }
  __device__ Off fstride() const { return Off(P) * P * P; }
};

__device__ __forceinline__ int bc_wrap(int i, int n, int lo, int hi) {
  if (i < 0) return lo == 0 ? i + n : 0;
  if (i >= n) return hi == 0 ? i - n : n - 1;
  return i;
}

template <typename T, typename OffT = int64_t>
struct LevelSource {
  using Off = OffT;  // unsigned int only for levels of fewer than 2^32 elements
  const T* base;  // the level storage [G][5][16^3]
  LevelGeom geo;
  int gx, gy, gz;
  __device__ Off col(int x, int y) const {
    const int X = bc_wrap(gx * 16 + x, geo.ngx * 16, geo.bc[0], geo.bc[1]);
    const int Y = bc_wrap(gy * 16 + y, geo.ngy * 16, geo.bc[2], geo.bc[3]);
    return Off((Y >> 4) * geo.ngx + (X >> 4)) * (5 * 4096) + (Y & 15) * 16 + (X & 15);
  }
  __device__ Off plane(int z) const {
    const int Z = bc_wrap(gz * 16 + z, geo.ngz * 16, geo.bc[4], geo.bc[5]);
    return Off(Z >> 4) * geo.ngx * geo.ngy * (5 * 4096) + (Z & 15) * 256;
  }
  __device__ Off fstride() const { return 4096; }
};

// kI: an interior column (x and y inside the group for every lane).
template <bool kI, typename T, class Src>
__device__ __forceinline__ void load_cons(const Src& src, typename Src::Off col, int z, T U[5]) {
  const typename Src::Off o = col + src.plane(z);
  const typename Src::Off fs = src.fstride();
#pragma unroll
  for (int q = 0; q < 5; ++q) U[q] = src.base[o + q * fs];
}

// A group of an AMR level: cells of the group and of the siblings around it
// are read from the level's states, cells where no sibling is from the
// group's scratch cells (interpolated there beforehand, only those).  A
// column's "offset" holds its coordinates, (y + 2) * 32 + (x + 2), clamped
// where the domain ends with outflow, as z is at the load, and above them its
// place in a plane of the scratch cells and whether it is one of the group's.
template <typename T>
struct AmrSource {
  using Off = unsigned int;
  const T* U;          // states of the level
  const T* shell;      // this group's scratch cells (shell_cell)
  const int* sib;      // LDS: sibling groups, [z][y][x] class (below, in, above), -1 where absent
  int below, self, above;  // sib of the centre column
  unsigned out;        // bits x-, x+, y-, y+, z-, z+: the group touches an outflow face of the domain
  static __device__ __forceinline__ int clamp(int i, unsigned lo, unsigned hi) {
    return (i < 0 && lo) ? 0 : (i > 15 && hi) ? 15 : i;
  }
  __device__ Off col(int x, int y) const {
    const int xc = clamp(x, out & 1u, out & 2u), yc = clamp(y, out & 4u, out & 8u);
    return unsigned(shell_in(xc, yc)) << 18 | shell_column(xc, yc) << 10 | unsigned((yc + 2) * 32 + xc + 2);
  }
};
template <bool kI, typename T>
__device__ __forceinline__ void load_cons(const AmrSource<T>& src, unsigned int col, int z, T U[5]) {
  const int zc = AmrSource<T>::clamp(z, src.out & 16u, src.out & 32u);
  const int x = int(col & 31u) - 2, y = int((col >> 5) & 31u) - 2, cz = (zc + 16) >> 4;
  const unsigned in = unsigned((zc & 15) * 256 + (y & 15) * 16 + (x & 15));
  // members read before they are selected from: a select of their addresses
  // would keep the source in memory
  const T *Us = src.U, *shell = src.shell;
  if constexpr (kI) {
    const int s0 = src.below, s1 = src.self, s2 = src.above;
    const int s = cz == 0 ? s0 : cz == 1 ? s1 : s2;  // uniform
    const T* b = s >= 0 ? Us + int64_t(s) * (5 * 4096) : shell;
    const unsigned o = s >= 0 ? in : unsigned(y * 16 + x) + shell_plane(true, zc);
    const unsigned fs = s >= 0 ? 4096u : unsigned(kShellCells);
#pragma unroll
    for (int q = 0; q < 5; ++q) U[q] = b[o + q * fs];
  } else {
    const int s = src.sib[cz * 9 + ((y + 16) >> 4) * 3 + ((x + 16) >> 4)];
    const unsigned at = ((col >> 10) & 255u) + ((col >> 18) != 0 ? shell_plane(true, zc) : shell_plane(false, zc));
    const T* b = s >= 0 ? Us + (int64_t(s) * (5 * 4096) + in) : shell + at;
    const unsigned fs = s >= 0 ? 4096u : unsigned(kShellCells);
#pragma unroll
    for (int q = 0; q < 5; ++q) U[q] = b[q * fs];
  }
}

template <bool kI, typename T, class Src>
__device__ __forceinline__ void load_prim(const Src& src, typename Src::Off col, int z, const Gas<T>& g, T W[5]) {
  T U[5];
  load_cons<kI>(src, col, z, U);
  cons_to_prim(U, g, W);
}

// LDS of one group's march.  kL pads the rows of the primitive and state
// tiles by kL elements (an LDS-layout option of the launch shapes: the same
// values at other addresses, so results are bit-identical).
template <typename T, int kL = 0>
struct Smem {
  static constexpr int PW = kPW + kL, SW = kSW + kL;
  static __device__ __forceinline__ int pi(int x, int y) { return (y + 2) * PW + (x + 2); }
  static __device__ __forceinline__ int si(int x, int y) { return (y + 1) * SW + (x + 1); }
  T P[5][PW * PW];       // primitive plane k
  T S[2][5][SW * SW];    // x+ and y+ half-step states of plane k
  T F[2][5][17 * 16];    // x and y fluxes of plane k
  T H[5][32];            // high-side states of the last faces: x = 16 (slot y), y = 16 (slot 16 + x)
};

// ------------------------------------------------------------- schemes ----
// The march computes one of two families of MHM + PLM steps:
//   DefaultScheme  generalized minmod on primitive variables and HLLC (the
//                  limiter specialized in its own inlined copy, see
//                  process_group), with the optional branch record;
//   ExtSchemeT     any MHM + PLM word of the other options (ExtOpts:
//                  generalized minmod, van Leer, van Albada or hybrid limiter,
//                  on primitive or characteristic variables; HLLC, Roe or
//                  HLLE; either wave-speed option; first order): the same
//                  half step with the slopes of ext_slopes and the fluxes of
//                  riemann_any.
struct DefaultScheme {};
// kChr (0 / 1) fixes the characteristic projection at compile time, kRoe
// the solver family (1: Roe, 0: HLLC or HLLE) and kLim the limiter of a
// second-order step (0 .. 3) or a first-order one (kFirstOrder); -1 leaves it
// to run time.  Each fixed combination is its own inlined copy, which carries
// only the registers of its own options.
constexpr int kFirstOrder = 4;
template <int kChr = -1, int kRoe = -1, int kLim = -1>
struct ExtSchemeT {
  ExtOpts o;
  __device__ __forceinline__ ExtOpts opts() const {
    ExtOpts r = o;
    if (kChr >= 0) r.chr = kChr;
    if (kRoe == 1) r.solver = 1;
    if (kRoe == 0) r.solver = o.solver == 2 ? 2 : 0;
    if (kLim >= 0) {
      r.lim = kLim;
      r.first_order = kLim == kFirstOrder;
    }
    return r;
  }
};

template <typename T>
__device__ __forceinline__ void scheme_half_step(const DefaultScheme&, const T Wc[5], const T Wn[3][2][5],
                                                 const Gas<T>& g, bool first_order, T Ut[3][2][5], unsigned* rec) {
  hancock_states(Wc, Wn, g, first_order, Ut, rec);
}

// The half step with full limited slopes s: face states Wc -+ s/2 (as the
// oracle's face values), then hancock_states' conserved form, fluxes and
// flux differences.
template <typename T, int kChr, int kRoe, int kLim>
__device__ __forceinline__ void scheme_half_step(const ExtSchemeT<kChr, kRoe, kLim>& sch, const T Wc[5], const T Wn[3][2][5],
                                                 const Gas<T>& g, bool, T Ut[3][2][5], unsigned*) {
  const ExtOpts o = sch.opts();
  T sum[5];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    T sl[5];
    if (o.first_order) {
#pragma unroll
      for (int q = 0; q < 5; ++q) sl[q] = T(0);
    } else if (d == 0) {
      ext_slopes<0>(Wn[0][0], Wc, Wn[0][1], g, o, sl);
    } else if (d == 1) {
      ext_slopes<1>(Wn[1][0], Wc, Wn[1][1], g, o, sl);
    } else {
      ext_slopes<2>(Wn[2][0], Wc, Wn[2][1], g, o, sl);
    }
    T dF[5];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      T W[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) W[q] = side == 0 ? Wc[q] - T(0.5) * sl[q] : Wc[q] + T(0.5) * sl[q];
      T* U = Ut[d][side];
      U[0] = W[0];
      U[1] = W[0] * W[1];
      U[2] = W[0] * W[2];
      U[3] = W[0] * W[3];
      U[4] = W[4] * g.inv_gm1 + T(0.5) * W[0] * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]);
      const T un = W[1 + d];
      T F[5];
      F[0] = U[0] * un;
      F[1] = U[1] * un;
      F[2] = U[2] * un;
      F[3] = U[3] * un;
      F[1 + d] = F[1 + d] + W[4];
      F[4] = (U[4] + W[4]) * un;
#pragma unroll
      for (int q = 0; q < 5; ++q) dF[q] = side == 0 ? F[q] : dF[q] - F[q];
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) sum[q] = d == 0 ? dF[q] : sum[q] + dF[q];
  }
#pragma unroll
  for (int q = 0; q < 5; ++q) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      Ut[d][0][q] = fma_(g.half_dtdx, sum[q], Ut[d][0][q]);
      Ut[d][1][q] = fma_(g.half_dtdx, sum[q], Ut[d][1][q]);
    }
  }
}

template <int D, typename T>
__device__ __forceinline__ bool scheme_flux(const DefaultScheme&, const T L[5], const T R[5], const Gas<T>& g, int ws,
                                            T F[5], unsigned* rec) {
  return hllc_flux<D>(L, R, g, ws, F, rec);
}
template <int D, typename T, int kChr, int kRoe, int kLim>
__device__ __forceinline__ bool scheme_flux(const ExtSchemeT<kChr, kRoe, kLim>& sch, const T L[5], const T R[5],
                                            const Gas<T>& g, int, T F[5], unsigned*) {
  return riemann_any<D>(L, R, g, sch.opts(), F);
}
// Two faces (normal axes D0, D1) at once; the default scheme interleaves
// their solves.
template <int D0, int D1, typename T>
__device__ __forceinline__ int scheme_flux2(const DefaultScheme&, const T L0[5], const T R0[5], const T L1[5],
                                            const T R1[5], const Gas<T>& g, int ws, T F0[5], T F1[5], unsigned* rec) {
  return hllc_flux2<D0, D1>(L0, R0, L1, R1, g, ws, F0, F1, rec);
}
template <int D0, int D1, typename T, int kChr, int kRoe, int kLim>
__device__ __forceinline__ int scheme_flux2(const ExtSchemeT<kChr, kRoe, kLim>& sch, const T L0[5], const T R0[5],
                                            const T L1[5], const T R1[5], const Gas<T>& g, int, T F0[5], T F1[5],
                                            unsigned*) {
  const ExtOpts o = sch.opts();
  return int(riemann_any<D0>(L0, R0, g, o, F0)) + int(riemann_any<D1>(L1, R1, g, o, F1));
}

// ---------------------------------------------------- one patch group ----
// Workgroup of 256 threads (4 waves; the hardware gives each wave of a
// workgroup its own SIMD).  Every thread owns one interior (x, y) column; the
// 64 threads of wave 0 also own one "halo" column one cell outside the
// interior (x = -1, x = 16, y = -1, y = 16), whose half-step states feed the
// faces on the group boundary, together with the column two cells out and,
// for 4 of them, an edge column (both only read as neighbours).  Wave 0 runs
// its halo role after its interior role in every phase; wave 2 solves the 32
// faces on the high x and y boundary of the group (their high-side states
// come from the halo role through LDS) after its own faces.

// The planes [lo, hi) of the group a workgroup completes: all of them, or one
// z segment (the march then runs the planes lo - 1 .. hi, recomputing the
// states of one plane beyond each end; the face between two segments is
// solved by both and counted by the upper one).
struct ZAll {
  static constexpr int lo = 0, hi = 16;
};
struct ZPart {
  int lo, hi;
};

// Per-column state of one role across the z-march.
template <typename T, bool kInterior, typename Off>
struct FwdCol {
  int cx, cy;
  bool xface16, yface16;  // halo columns at x = 16 / y = 16 (high side of the last x / y face)
  Off col;
  T Wm[5], Wc[5], Wp[5];  // primitive states at planes k-1, k, k+1
  T Un[5];                // conserved values of the next plane to convert (in flight)
  T Ux[5], Uy[5];         // own x- and y- face states of plane k (interior)
  T Uz[5], Fz0[5];        // interior: z+ face state of plane k-1; z flux at the low face of plane k-1
};

template <typename T, bool kI, class Src, class Z>
__device__ __forceinline__ void fwd_col_init(FwdCol<T, kI, typename Src::Off>& c, const Src& src, int cx, int cy, const Gas<T>& gas, const Z& zr) {
  c.cx = cx;
  c.cy = cy;
  c.xface16 = !kI && cx == 16;
  c.yface16 = !kI && cy == 16;
  c.col = src.col(cx, cy);
  if (kI) load_prim<kI>(src, c.col, zr.lo - 2, gas, c.Wm);
  load_prim<kI>(src, c.col, zr.lo - 1, gas, c.Wc);
  load_cons<kI>(src, c.col, zr.lo, c.Un);
}

// Next plane of the column (prefetched one iteration ahead); publish plane k.
template <typename T, bool kI, class Src, int kL, class Z>
__device__ __forceinline__ void fwd_col_publish(FwdCol<T, kI, typename Src::Off>& c, const Src& src, int k, const Gas<T>& gas,
                                                Smem<T, kL>& sm, const Z& zr) {
  const int zhi = kI ? zr.hi + 1 : zr.hi;  // last plane of the column that is read
  // Convert the plane that arrived, then issue the next one.  The load is
  // unconditional (plane index clamped to the column's last plane, re-read
  // harmlessly near the top) and issued after the conversion, so the loaded
  // registers are never merged with old values: a merge would need the data
  // and wait for the load that is meant to stay in flight.
  cons_to_prim(c.Un, gas, c.Wp);
  asm volatile("" ::: "memory");
  load_cons<kI>(src, c.col, k + 2 <= zhi ? k + 2 : zhi, c.Un);
#pragma unroll
  for (int q = 0; q < 5; ++q) sm.P[q][sm.pi(c.cx, c.cy)] = c.Wc[q];
}

// CFL signal-speed maxima of a group live in LDS as [z half][patch xy][64
// columns of the patch] (the order the epilogue reduces in): a thread's slot
// for z half 0 is cfl_slot(tid), its slot for z half 1 lies kCflHalfStride
// doubles further.  Kept in LDS rather than registers (4 VGPRs fewer through
// the march).
constexpr int kCflHalfStride = 256;
__device__ __forceinline__ int cfl_slot(int tid) {
  const int x = tid & 15, y = tid >> 4;
  return ((y >> 3) * 2 + (x >> 3)) * 64 + (y & 7) * 8 + (x & 7);
}

// Half-step face states of the column's state cell at plane k.  Interior
// columns also solve the z-face k-1/2 and complete plane k-1.
template <typename T, bool kI, class Src, int kL, class Sch, class Z>
__device__ __forceinline__ int fwd_col_states(const Sch& sch, FwdCol<T, kI, typename Src::Off>& c, const Src& src, T* __restrict__ out, int k,
                                              const Gas<T>& gas, int first_order, int ws, Smem<T, kL>& sm, double* smax,
                                              double gamma_d, T* __restrict__ ff, unsigned* rec, const Z& zr, unsigned ff_planes) {
  const int cx = c.cx, cy = c.cy;
  int bad = 0;
  // What the update of plane k-1 at the end of this phase takes.  The default
  // scheme has both early; the other words fetch them where they are used, since
  // their solves need the registers (FP64 spills of the HLLC / Roe copies 6 / 28
  // -> 0 / 9, 2048 groups 16% faster on average; only the differences late: 0 /
  // 17 and 13%).
  constexpr bool kEarly = std::is_same<Sch, DefaultScheme>::value;
  // U^n of plane k-1, issued first so that the load's latency overlaps the
  // half step and the z-face solve
  T Uold[5];
  if (kEarly && kI && k > zr.lo) load_cons<kI>(src, c.col, k - 1, Uold);
  // x/y flux differences of plane k-1 (fluxes written last iteration)
  T acc[5];
  if (kEarly && kI && k > zr.lo) {
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      acc[q] = sm.F[0][q][fxidx(cx + 1, cy)] - sm.F[0][q][fxidx(cx, cy)];
      acc[q] = acc[q] + (sm.F[1][q][fyidx(cx, cy + 1)] - sm.F[1][q][fyidx(cx, cy)]);
    }
  }
  if (!kI && (k < zr.lo || k >= zr.hi)) return 0;
  T Wn[3][2][5];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    Wn[0][0][q] = sm.P[q][sm.pi(cx - 1, cy)];
    Wn[0][1][q] = sm.P[q][sm.pi(cx + 1, cy)];
    Wn[1][0][q] = sm.P[q][sm.pi(cx, cy - 1)];
    Wn[1][1][q] = sm.P[q][sm.pi(cx, cy + 1)];
    Wn[2][0][q] = c.Wm[q];
    Wn[2][1][q] = c.Wp[q];
  }
  T Ut[3][2][5];
  scheme_half_step(sch, c.Wc, Wn, gas, first_order != 0, Ut, rec);
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    sm.S[0][q][sm.si(cx, cy)] = Ut[0][1][q];
    sm.S[1][q][sm.si(cx, cy)] = Ut[1][1][q];
    if (kI) {
      c.Ux[q] = Ut[0][0][q];
      c.Uy[q] = Ut[1][0][q];
    }
  }
  // halo columns at x = 16 / y = 16: their low x / y state is the high side
  // of the last face, solved by another wave after the next barrier
  if (!kI && (c.xface16 || c.yface16)) {
    const int slot = c.xface16 ? cy : 16 + cx;
#pragma unroll
    for (int q = 0; q < 5; ++q) sm.H[q][slot] = c.xface16 ? Ut[0][0][q] : Ut[1][0][q];
  }
  if (kI) {
    if (k >= zr.lo) {
      T Fz1[5];
      const int bz = scheme_flux<2>(sch, c.Uz, Ut[2][0], gas, ws, Fz1, rec);
      if (!kEarly && k > zr.lo) load_cons<kI>(src, c.col, k - 1, Uold);
      bool own = true;
      if constexpr (!std::is_same<Z, ZAll>::value) own = k < zr.hi || zr.hi == 16;
      bad += own ? bz : 0;
      if (ff != nullptr && (k & 7) == 0 && own && ((ff_planes >> (6 + (k >> 3))) & 1u)) {
        // z faces on a patch boundary (z = 0, 8, 16): plane 6 + k/8, entry y*16 + x
        T* o = ff + (6 + (k >> 3)) * 5 * 256 + cy * 16 + cx;
#pragma unroll
        for (int q = 0; q < 5; ++q) o[q * 256] = Fz1[q];
      }
      if (k > zr.lo) {
        if (!kEarly) {
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            acc[q] = sm.F[0][q][fxidx(cx + 1, cy)] - sm.F[0][q][fxidx(cx, cy)];
            acc[q] = acc[q] + (sm.F[1][q][fyidx(cx, cy + 1)] - sm.F[1][q][fyidx(cx, cy)]);
          }
        }
        // complete plane k-1: U^{n+1} = U^n - dt/dx [(x) + (y) + (z)]
        T Un[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          const T a = acc[q] + (Fz1[q] - c.Fz0[q]);
          Un[q] = Uold[q] - gas.dtdx * a;
          out[q * 4096 + ((k - 1) * 16 + cy) * 16 + cx] = Un[q];
        }
        bad += unphysical(Un, gas);
        if (smax != nullptr) {
          const double s = cfl_signal_speed(double(Un[0]), double(Un[1]), double(Un[2]), double(Un[3]),
                                            double(Un[4]), gamma_d);
          double& m = smax[((k - 1) >> 3) * kCflHalfStride];
          if (s > m) m = s;
        }
      }
#pragma unroll
      for (int q = 0; q < 5; ++q) c.Fz0[q] = Fz1[q];
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) c.Uz[q] = Ut[2][1][q];
  }
  return bad;
}

// x and y faces of plane k that an interior column solves: its low x and low
// y face.
template <typename T, bool kI, typename Off, int kL, class Sch, class Z>
__device__ __forceinline__ int fwd_col_faces(const Sch& sch, FwdCol<T, kI, Off>& c, int k, const Gas<T>& gas, int ws, Smem<T, kL>& sm,
                                             unsigned* rec, const Z& zr) {
  if (!kI || k < zr.lo || k >= zr.hi) return 0;
  const int cx = c.cx, cy = c.cy;
  T Lx[5], Fx[5], Ly[5], Fy[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    Lx[q] = sm.S[0][q][sm.si(cx - 1, cy)];
    Ly[q] = sm.S[1][q][sm.si(cx, cy - 1)];
  }
  const int bad = scheme_flux2<0, 1>(sch, Lx, c.Ux, Ly, c.Uy, gas, ws, Fx, Fy, rec);
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    sm.F[0][q][fxidx(cx, cy)] = Fx[q];
    sm.F[1][q][fyidx(cx, cy)] = Fy[q];
  }
  return bad;
}

// Patch-boundary face fluxes of plane k from the flux arrays: axis 0 the x
// faces at x = 0, 8, 16 (plane x/8 of ff, entry z*16 + y), axis 1 the y faces at
// y = 0, 8, 16 (plane 3 + y/8, entry x*16 + z).  One wave copies an axis, in the
// next plane's first phase: the plain waves 1 and 3, which the others wait
// for least.  The y planes run along z, so a plane of the march holds one
// entry of each of their rows: up to 8 planes wait in LDS (stage, kFluxStage
// elements) and are stored together.  Stored by the threads that solve the
// faces, a few lanes of every wave at a time, the fluxes cost a third of the
// step (AMR level step 694 us against 521 without fluxes; by one wave per
// axis 641, staged 586).
constexpr int kFluxStage = 8 * 240;
template <typename T, int kL>
__device__ __forceinline__ void put_face_fluxes(int axis, int lane, int k, bool last, int first, const Smem<T, kL>& sm,
                                                T* __restrict__ ff, T* stage, unsigned planes) {
  planes >>= 3 * axis;
  if ((planes & 7u) == 0) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int v = j * 64 + lane, pq = v >> 4, i = v & 15;  // pq = 5 (coordinate / 8) + field
    if (v >= 240) break;
    const int p = pq / 5, q = pq - 5 * p;
    if (!((planes >> p) & 1u)) continue;
    if (axis == 0) ff[pq * 256 + k * 16 + i] = sm.F[0][q][fxidx(8 * p, i)];
    else stage[(k & 7) * 240 + v] = sm.F[1][q][fyidx(i, 8 * p)];
  }
  if (axis == 1 && ((k & 7) == 7 || last)) {
    // planes k0 .. k of each row (the same lane stored them)
    const int k0 = (k & 8) > first ? (k & 8) : first;
    for (int v = lane; v < 240; v += 64) {
      if (!((planes >> ((v >> 4) / 5)) & 1u)) continue;
      T* o = ff + (15 + (v >> 4)) * 256 + (v & 15) * 16;
      for (int z = k0; z <= k; ++z) o[z] = stage[(z & 7) * 240 + v];
    }
  }
}

// The 32 last faces of plane k (x = 16 for lanes 0..15 at y = lane, y = 16
// for lanes 16..31 at x = lane - 16), in one solver pass: a y face is solved
// in the x-normal frame with its states rotated (m_y, m_z, m_x) -> (m_x,
// m_y, m_z), the same arithmetic on the same values as the y-normal solver,
// and the flux rotated back.  The halo wave wrote the high-side states to
// H; this pass runs on another wave, which has no halo work.
template <typename T, int kL, class Sch, class Z>
__device__ __forceinline__ int last_faces(const Sch& sch, int lane, int k, const Gas<T>& gas, int ws, Smem<T, kL>& sm,
                                          unsigned* rec, const Z& zr) {
  if (k < zr.lo || k >= zr.hi || lane >= 32) return 0;
  const bool yf = lane >= 16;
  const int i = lane & 15;
  const T* Sb = yf ? &sm.S[1][0][sm.si(i, 15)] : &sm.S[0][0][sm.si(15, i)];
  T L[5], R[5], Lr[5], Rr[5], F[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    L[q] = Sb[q * sm.SW * sm.SW];
    R[q] = sm.H[q][lane];
  }
  Lr[0] = L[0];
  Lr[1] = yf ? L[2] : L[1];
  Lr[2] = yf ? L[3] : L[2];
  Lr[3] = yf ? L[1] : L[3];
  Lr[4] = L[4];
  Rr[0] = R[0];
  Rr[1] = yf ? R[2] : R[1];
  Rr[2] = yf ? R[3] : R[2];
  Rr[3] = yf ? R[1] : R[3];
  Rr[4] = R[4];
  const int bad = scheme_flux<0>(sch, Lr, Rr, gas, ws, F, rec);
  T* Fb = yf ? &sm.F[1][0][fyidx(i, 16)] : &sm.F[0][0][fxidx(16, i)];
  Fb[0] = F[0];
  Fb[1 * 17 * 16] = yf ? F[3] : F[1];
  Fb[2 * 17 * 16] = yf ? F[1] : F[2];
  Fb[3 * 17 * 16] = yf ? F[2] : F[3];
  Fb[4 * 17 * 16] = F[4];
  return bad;
}

template <typename T, bool kI, typename Off>
__device__ __forceinline__ void fwd_col_shift(FwdCol<T, kI, Off>& c) {
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    c.Wm[q] = c.Wc[q];
    c.Wc[q] = c.Wp[q];
  }
}

// Roles of the waves of a workgroup beyond their interior columns.
enum WaveRole { kRoleHalo = 0, kRoleLastFaces = 1, kRolePlain = 2 };

// The z-march of one wave: interior role, plus the halo roles (kRoleHalo,
// wave 0) or the solve of the 32 last faces (kRoleLastFaces, wave 2).  Every
// instantiation passes the same barriers in the same order.
template <typename T, class Src, int kRole, int kUnroll, int kL, class Sch, class Z>
__device__ __forceinline__ int march_group(const Sch& sch, const Src& src, T* __restrict__ out, const Gas<T>& gas, int first_order,
                                           int ws, Smem<T, kL>& sm, double* smax, double gamma_d, int tid,
                                           T* __restrict__ ff, unsigned* rec, const Z& zr, T* ff_stage, unsigned ff_planes) {
  // halo role: side 0..3 = x-, x+, y-, y+; the column two cells out; lanes
  // 0..3 also one of the 4 edge columns
  const int lane = tid & 63;
  const int side = lane >> 4, kk = lane & 15;
  const int hx = side == 0 ? -1 : side == 1 ? 16 : kk, hy = side == 2 ? -1 : side == 3 ? 16 : kk;
  const int ox = side == 0 ? -2 : side == 1 ? 17 : kk, oy = side == 2 ? -2 : side == 3 ? 17 : kk;
  const int ex = (lane & 1) ? 16 : -1, ey = (lane & 2) ? 16 : -1;
  constexpr bool kHalo = kRole == kRoleHalo;
  const bool has_edge = kHalo && lane < 4;

  using Off = typename Src::Off;
  FwdCol<T, true, Off> ci;
  FwdCol<T, false, Off> ch;
  fwd_col_init(ci, src, tid & 15, tid >> 4, gas, zr);
  Off col_out = 0, col_edge = 0;
  T Uo[5], Ue[5];  // halo role: 2-deep and edge column, plane k (in flight)
  if (kHalo) {
    col_out = src.col(ox, oy);
    col_edge = src.col(has_edge ? ex : ox, has_edge ? ey : oy);  // lanes without an edge re-read their 2-deep column
    fwd_col_init(ch, src, hx, hy, gas, zr);
    load_cons<false>(src, col_out, zr.lo, Uo);
    load_cons<false>(src, col_edge, zr.lo, Ue);
  }
  int bad = 0;

#pragma unroll kUnroll
  for (int k = zr.lo - 1; k <= zr.hi; ++k) {
    // ---- next planes (prefetched); publish plane k to LDS
    fwd_col_publish(ci, src, k, gas, sm, zr);
    if (kHalo) {
      fwd_col_publish(ch, src, k, gas, sm, zr);
      // 2-deep and edge columns (planes lo..hi-1; loads clamped, no merge of
      // loaded registers with old values)
      T Wo[5], We[5];
      cons_to_prim(Uo, gas, Wo);
      cons_to_prim(Ue, gas, We);
      asm volatile("" ::: "memory");
      const int kn = k + 1 < zr.lo ? zr.lo : (k + 1 >= zr.hi ? zr.hi - 1 : k + 1);
      load_cons<false>(src, col_out, kn, Uo);
      load_cons<false>(src, col_edge, kn, Ue);
      if (k >= zr.lo && k < zr.hi) {
#pragma unroll
        for (int q = 0; q < 5; ++q) sm.P[q][sm.pi(ox, oy)] = Wo[q];
        if (has_edge) {
#pragma unroll
          for (int q = 0; q < 5; ++q) sm.P[q][sm.pi(ex, ey)] = We[q];
        }
      }
    }
    __syncthreads();

    // ---- half-step face states of plane k; z-face and update of plane k-1
    if (kRole == kRolePlain && ff != nullptr && k > zr.lo)
      put_face_fluxes(tid >> 7, lane, k - 1, k == zr.hi, zr.lo, sm, ff, ff_stage, ff_planes);
    bad += fwd_col_states(sch, ci, src, out, k, gas, first_order, ws, sm, smax, gamma_d, ff, rec, zr, ff_planes);
    if (kHalo) bad += fwd_col_states(sch, ch, src, out, k, gas, first_order, ws, sm, nullptr, gamma_d, (T*)nullptr, rec, zr, ff_planes);
    __syncthreads();

    // ---- x and y faces of plane k
    bad += fwd_col_faces(sch, ci, k, gas, ws, sm, rec, zr);
    if (kRole == kRoleLastFaces) bad += last_faces(sch, lane, k, gas, ws, sm, rec, zr);

    fwd_col_shift(ci);
    if (kHalo) fwd_col_shift(ch);
  }
  return bad;
}

// Advance one group: read through `src`, write the 16^3 x 5 interior to `out`
// (field stride 4096).  Returns this thread's unphysical count.  If smax is
// non-null (the thread's cfl_slot in an LDS array, both halves set to 0),
// also leaves there the maximum CFL signal speed of the thread's interior
// cells in patch-z halves 0..7 and 8..15.  If ff is non-null, also writes the
// fluxes of the faces on the patch boundaries (normal coordinate 0, 8, 16 of
// each axis) to ff as [9][5][256]: plane 3 axis + k holds the faces at 8 k,
// entry b * 16 + a with (a, b) the transverse coordinates in cyclic order
// (the flux registers of coarse-fine coupling); ff_stage: kFluxStage elements of
// LDS for it; ff_planes: bit 3 axis + k set for the planes to write.  `tid` is the thread's index in the
// workgroup (a loop over groups passes it opaque, so that the compiler keeps
// thread-derived addresses out of the loop's live set).  Wave 0 runs the
// march with the halo roles, wave 2 with the last faces, waves 1 and 3 with
// their interior columns only (wave-uniform branches).  Two co-resident
// workgroups get their waves on SIMDs (0, 2, 1, 3) and (2, 1, 3, 0), so the
// halo waves sit on SIMDs 0 and 2 and the last-face waves on SIMDs 1 and 3.
// The second-order scheme (first_order == 0) gets its own inlined copies
// with the limiter unconditional; the first-order one keeps the runtime flag.
// kPrio: the halo wave (the most work per plane) and the last-faces wave take
// issue priority over the plain waves they share a SIMD with, so the plane's
// barrier is reached sooner.  Measured on the 256^3 shear layer: with four
// waves per SIMD (FP32, high occupancy) the step is 6-8% faster; with two
// (FP64, FP32 low occupancy) 2-5% slower, so those kernels keep equal
// priorities.
template <typename T, bool kPrio, class Src, int kL, class Sch, class Z>
__device__ __forceinline__ int march_roles(const Sch& sch, const Src& src, T* __restrict__ out, const Gas<T>& gas,
                                           int first_order, int ws, Smem<T, kL>& sm, double* smax, double gamma_d,
                                           int tid, T* __restrict__ ff, unsigned* rec, const Z& zr, T* ff_stage,
                                           unsigned ff_planes) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Two planes per loop iteration, so that the register rotation of a
  // column's planes (Wm <- Wc <- Wp, z-face state and flux) becomes renaming
  // instead of moves (2-3% fewer VALU instructions per plane): every role in
  // FP32 at the low occupancy target (step 2% faster), the plain and
  // last-faces roles in FP64 (step 0.5-0.8% faster; the halo role, which
  // carries a second column, would need more than 256 VGPRs).  The four-wave
  // FP32 kernels (kPrio; 128 VGPRs, where it spills) and the other scheme
  // words keep one plane.
  constexpr int kU = (sizeof(T) == 4 && !kPrio) ? 2 : 1;   // halo role
  constexpr int kU2 = !kPrio ? 2 : 1;                       // the other roles
  if constexpr (kPrio) {
    if (wave == 0) __builtin_amdgcn_s_setprio(2);
    if (wave == 2) __builtin_amdgcn_s_setprio(1);
  }
  if constexpr (std::is_same<Z, ZPart>::value) {
    // a z segment: few planes, one per loop iteration, one copy
    if (wave == 0) return march_group<T, Src, kRoleHalo, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    if (wave == 2)
      return march_group<T, Src, kRoleLastFaces, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    return march_group<T, Src, kRolePlain, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
  } else if constexpr (!std::is_same<Sch, DefaultScheme>::value) {
    // the other words: one copy (their options are run-time anyway), one
    // plane per loop iteration
    if (wave == 0) return march_group<T, Src, kRoleHalo, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    if (wave == 2)
      return march_group<T, Src, kRoleLastFaces, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    return march_group<T, Src, kRolePlain, 1>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
  } else {
    if (first_order == 0) {
      if (wave == 0) return march_group<T, Src, kRoleHalo, kU>(sch, src, out, gas, 0, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
      if (wave == 2)
        return march_group<T, Src, kRoleLastFaces, kU2>(sch, src, out, gas, 0, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
      return march_group<T, Src, kRolePlain, kU2>(sch, src, out, gas, 0, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    }
    if (wave == 0)
      return march_group<T, Src, kRoleHalo, kU>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    if (wave == 2)
      return march_group<T, Src, kRoleLastFaces, kU2>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
    return march_group<T, Src, kRolePlain, kU2>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, rec, zr, ff_stage, ff_planes);
  }
}

// rec_out (diagnostic, optional): the group's branch record -- every
// thread's decisions hashed in its own order (record()), the threads' hashes
// combined by XOR, which is independent of the order they arrive in.
template <typename T, bool kPrio, class Src, int kL, class Sch = DefaultScheme, class Z = ZAll>
__device__ __forceinline__ int process_group(const Src& src, T* __restrict__ out, const Gas<T>& gas,
                                             int first_order, int ws, Smem<T, kL>& sm, double* smax,
                                             double gamma_d, int tid = threadIdx.x, T* __restrict__ ff = nullptr,
                                             unsigned* __restrict__ rec_out = nullptr, const Sch& sch = Sch(),
                                             const Z& zr = Z(), T* ff_stage = nullptr, unsigned ff_planes = 0x1ffu) {
  if (rec_out == nullptr)
    return march_roles<T, kPrio>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, nullptr, zr, ff_stage, ff_planes);
  __shared__ unsigned grp_rec;
  if (tid == 0) grp_rec = 0u;  // the march's first barrier orders this before any XOR
  unsigned h = 2166136261u ^ (unsigned(tid) * 0x9E3779B9u);
  const int bad = march_roles<T, kPrio>(sch, src, out, gas, first_order, ws, sm, smax, gamma_d, tid, ff, &h, zr, ff_stage, ff_planes);
  atomicXor(&grp_rec, h);
  __syncthreads();
  if (tid == 0) *rec_out = grp_rec;
  return bad;
}

// Reduce the per-thread signal-speed maxima of one group (the LDS array
// `slots` of cfl_slot's layout, 512 doubles: patch p = (pz*2 + py)*2 + px owns
// slots [64 p, 64 p + 64)) to its 8 patch time-steps: thread p < 8 scans its
// patch's 64 slots (a maximum is exact in any order; NaN and negative speeds
// never win over the start value 0).  A butterfly of lane shuffles over the
// 4 waves (each wave two patches) was measured slower on the 256^3 step (FP64
// 0.904 vs 0.881 ms, FP32 0.553 vs 0.493 ms).  Stores dt_patch[p]
// (optional) and folds dt * fold_scale into *dt_min (optional; integer
// minimum of non-negative doubles: exact and order-independent).  half >= 0:
// only the patches of that z half (a workgroup that completed part of the
// group).  Every thread of the workgroup must call it.
__device__ __forceinline__ void cfl_epilogue(const double* slots, double c_cfl_dx,
                                             double* __restrict__ dt_patch, unsigned long long* __restrict__ dt_min,
                                             double fold_scale = 1.0, int tid = threadIdx.x, int half = -1) {
  __syncthreads();
  if (tid < 8 && (half < 0 || tid >> 2 == half)) {
    double m = 0.0;
    for (int i = 0; i < 64; ++i) {
      const double s = slots[tid * 64 + i];
      if (s > m) m = s;
    }
    const double dt = c_cfl_dx / m;
    if (dt_patch != nullptr) dt_patch[tid] = dt;
    if (dt_min != nullptr) atomicMin(dt_min, (unsigned long long)__double_as_longlong(dt * fold_scale));
  }
}

template <typename T>
__device__ __forceinline__ void set_dt(Gas<T>& gas, const double* dt_dev, double dx) {
  if (dt_dev != nullptr) {
    const double dt = *dt_dev;
    gas.dtdx = T(dt / dx);
    gas.half_dtdx = T(0.5 * (dt / dx));
  }
}

// Waves per SIMD the register allocation must allow.  Each wave of a 4-wave
// workgroup gets its own SIMD, so this is also the number of workgroups per
// CU the registers allow: FP64 2 (<= 256 VGPRs; two workgroups' LDS fits in
// 160 KB) or 1; FP32 4 (<= 128 VGPRs) or 2.  `value` is the padded step's.
template <typename T> struct MinWaves;
template <> struct MinWaves<double> { static constexpr int hi = 2, lo = 1; static constexpr int value = hi; };
template <> struct MinWaves<float> { static constexpr int hi = 4, lo = 2; static constexpr int value = hi; };

}  // namespace gh
