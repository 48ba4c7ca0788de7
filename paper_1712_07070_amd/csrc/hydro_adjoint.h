// Reverse-mode (vector-Jacobian) counterparts of the MHM step's device
// arithmetic in hydro_device.h.  Each *_vjp routine recomputes the forward
// intermediates it needs from the same inputs (so branch decisions -- limiter
// case, HLLC branch, min/max of wave speeds -- are taken exactly as in the
// forward pass) and returns the cotangents of its inputs given the cotangents
// of its outputs.
//
// Derivative conventions at non-smooth points (shared with the oracle's
// dual-number instantiation):
//   * limiter: zero when the one-sided differences are not strictly of one
//     sign; otherwise through the argument attaining the minimum, the first of
//     (theta|dm|, |dc|, theta|dp|) on ties; the sign factor has zero derivative;
//   * min/max of wave speeds: through the first argument unless the second is
//     strictly smaller/larger;
//   * HLLC: the derivative of the branch the forward pass took.
#pragma once

#include "hydro_device.h"

namespace gh {

// ----------------------------------------------- a1: cons -> primitive VJP --
// W = (rho, m/rho, p) with p = gm1 (E - (m.u)/2).  Given gW, add gU.
template <typename T>
__device__ __forceinline__ void cons_to_prim_vjp(const T U[5], const Gas<T>& g, const T gW[5], T gU[5]) {
  const T inv = Fp<T>::rcp(U[0]);
  const T u = U[1] * inv, v = U[2] * inv, w = U[3] * inv;
  const T gp = gW[4] * g.gm1;
  // p = gm1 (E - (m_x u + m_y v + m_z w)/2): dp/dm_i = -gm1 u_i, dp/drho = gm1 |u|^2 / 2
  gU[0] = gU[0] + gW[0] - (gW[1] * u + gW[2] * v + gW[3] * w) * inv + T(0.5) * gp * (u * u + v * v + w * w);
  gU[1] = gU[1] + gW[1] * inv - gp * u;
  gU[2] = gU[2] + gW[2] * inv - gp * v;
  gU[3] = gU[3] + gW[3] * inv - gp * w;
  gU[4] = gU[4] + gp;
}

// -------------------------------------------------- a2: limiter VJP -------
// h = half_slope(qm, q0, qp); given gh, add to gqm, gq0, gqp.
//   h = sgn * min(...) with sgn the common sign: h = half_theta*dm, (qp-qm)/4 or half_theta*dp
// Without branches: a wave whose lanes differ takes each of them in turn (the
// fused adjoint of 64 groups, FP32 269 -> 245 us, FP64 302 -> 285).  kBranch
// keeps them for the FP64 cells kernel, which spills more without (512 groups
// faces + cells 895 us, 1007 without).
template <bool kBranch, typename T>
__device__ __forceinline__ void half_slope_vjp(T qm, T q0, T qp, T half_theta, T gh, T& gqm, T& gq0, T& gqp) {
  const T dm = q0 - qm;
  const T dp = qp - q0;
  const bool on = dm * dp > T(0);
  if (kBranch && !on) return;
  const T a = half_theta * fabs_(dm);
  const T b = T(0.25) * fabs_(qp - qm);
  const T c = half_theta * fabs_(dp);
  // the argument attaining the minimum: dm (first), the central one, dp
  const bool mid = b < a;
  const bool last = c < (mid ? b : a);
  const bool first = !mid && !last;
  if (kBranch) {
    if (first) {
      gq0 = gq0 + half_theta * gh;
      gqm = gqm - half_theta * gh;
    } else if (!last) {
      gqp = gqp + T(0.25) * gh;
      gqm = gqm - T(0.25) * gh;
    } else {
      gqp = gqp + half_theta * gh;
      gq0 = gq0 - half_theta * gh;
    }
    return;
  }
  const T w = (mid && !last) ? T(0.25) : half_theta;
  gqm = (on && !last) ? gqm - w * gh : gqm;
  gqp = (on && !first) ? gqp + w * gh : gqp;
  const T s = first ? half_theta : -half_theta;
  gq0 = (on && (first || last)) ? gq0 + s * gh : gq0;
}

// ------------------------------------------- a3 + a4: Hancock states VJP ---
// Forward: hancock_states(Wc, Wn, g, first_order, Ut).  Streaming form: the
// neighbour states, the face-state cotangents and the neighbour outputs are
// reached through callbacks, one direction at a time, so that a caller can
// keep them in LDS and only one direction's values are live at once.
//   getW(d, side, T W[5])   primitive state of neighbour (d, side)
//   getG(d, side, T g[5])   cotangent gUt[d][side] (zero for unused faces)
//   putN(d, side, T g[5])   receives the cotangent of neighbour (d, side)
//   gWc                     receives the cotangent of the cell's own state
template <bool kBranch = false, typename T, class GetW, class GetG, class PutN>
__device__ __forceinline__ void hancock_states_vjp_stream(const T Wc[5], const Gas<T>& g, bool first_order,
                                                          GetW&& getW, GetG&& getG, PutN&& putN, T gWc[5]) {
  // dU = half_dtdx * sum_d (F_d(-) - F_d(+)); every face state receives dU
  T gdU[5] = {T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    T a[5], b[5];
    getG(d, 0, a);
    getG(d, 1, b);
#pragma unroll
    for (int q = 0; q < 5; ++q) gdU[q] = gdU[q] + (a[q] + b[q]);
  }
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    gdU[q] = g.half_dtdx * gdU[q];
    gWc[q] = T(0);
  }
  // the face cotangents are fetched again per direction below: keep the
  // compiler from holding all six vectors live across the loop
  asm volatile("" ::: "memory");
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    T Wl[5], Wr[5];
    getW(d, 0, Wl);
    getW(d, 1, Wr);
    T h[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) h[q] = first_order ? T(0) : half_slope(Wl[q], Wc[q], Wr[q], g.half_theta);
    T gh[5] = {T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const T sgn = side == 0 ? T(1) : T(-1);  // face flux enters dU with this sign
      T W[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) W[q] = side == 0 ? Wc[q] - h[q] : Wc[q] + h[q];
      const T rho = W[0], u = W[1], v = W[2], w = W[3], p = W[4];
      const T U1 = rho * u, U2 = rho * v, U3 = rho * w;
      const T U4 = p * g.inv_gm1 + T(0.5) * rho * (u * u + v * v + w * w);
      const T un = W[1 + d];
      T gUt[5];
      getG(d, side, gUt);
      // cotangent of this face state's conserved variables: direct + via its flux
      T gF[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) gF[q] = sgn * gdU[q];
      T gU[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) gU[q] = gUt[q] + gF[q] * un;
      // flux: F = U * un (+ p on the normal momentum), F4 = (U4 + p) un
      T gW[5] = {T(0), T(0), T(0), T(0), T(0)};
      gW[1 + d] = gF[0] * rho + gF[1] * U1 + gF[2] * U2 + gF[3] * U3 + gF[4] * (U4 + p);
      gW[4] = gF[1 + d] + gF[4] * un;
      // cons: U = (rho, rho u, rho v, rho w, p/gm1 + rho |u|^2 / 2)
      gW[0] = gW[0] + gU[0] + gU[1] * u + gU[2] * v + gU[3] * w + gU[4] * (T(0.5) * (u * u + v * v + w * w));
      gW[1] = gW[1] + gU[1] * rho + gU[4] * (rho * u);
      gW[2] = gW[2] + gU[2] * rho + gU[4] * (rho * v);
      gW[3] = gW[3] + gU[3] * rho + gU[4] * (rho * w);
      gW[4] = gW[4] + gU[4] * g.inv_gm1;
      // W_{d,-} = Wc - h, W_{d,+} = Wc + h
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        gWc[q] = gWc[q] + gW[q];
        gh[q] = side == 0 ? gh[q] - gW[q] : gh[q] + gW[q];
      }
    }
    T gl[5] = {T(0), T(0), T(0), T(0), T(0)}, gr[5] = {T(0), T(0), T(0), T(0), T(0)};
    if (!first_order) {
#pragma unroll
      for (int q = 0; q < 5; ++q)
        half_slope_vjp<kBranch>(Wl[q], Wc[q], Wr[q], g.half_theta, gh[q], gl[q], gWc[q], gr[q]);
    }
    putN(d, 0, gl);
    putN(d, 1, gr);
  }
}

// ---------------------------------------------------------- a5: HLLC VJP ---
// Forward: hllc_flux<D>(L, R, g, ws, F).  Given gF (axis frame), the
// cotangents of the two conserved input states.
//
// As in the forward solve only one side K enters the flux, as
// F_K + S (U*_K - U_K) with S = S_K in the star regions; beyond the fan S = 0
// and the divisors are 1, so that the same statements give the derivative of
// F_K, and the cotangents of S_K and S* are dropped.  The face solves and the
// limiter are the adjoint's arithmetic: with a branch per region and per side
// the lanes of a wave took the paths in turn (192^3 FP32 level adjoint 1.23
// ms, 1.11 with none; 128^3 FP64 607 -> 565 us); taking an x and a y face
// in turn statement by statement gave nothing more.  Where all lanes took one
// path the branches were the faster form: 512 groups FP64, noise and turbulence
// 677 -> 631 us, a shear layer 621 -> 630, a uniform or supersonic state 604 ->
// 630.  Tests of the whole wave around the star region and around the limiter
// bring those two to 588 and 611, but noise to 644 and the shear layer to 642.
template <int D, typename T>
__device__ __forceinline__ void hllc_flux_vjp(const T Lx[5], const T Rx[5], const Gas<T>& g, int ws, const T gFx[5],
                                              T gLx[5], T gRx[5]) {
  constexpr int n = 1 + D, t1 = 1 + (D + 1) % 3, t2 = 1 + (D + 2) % 3;
  // normal frame
  const T L[5] = {Lx[0], Lx[n], Lx[t1], Lx[t2], Lx[4]}, R[5] = {Rx[0], Rx[n], Rx[t1], Rx[t2], Rx[4]};
  const T gF[5] = {gFx[0], gFx[n], gFx[t1], gFx[t2], gFx[4]};
  // ---- forward recomputation
  const T iL = Fp<T>::rcp(L[0]);
  const T iR = Fp<T>::rcp(R[0]);
  const T uL = L[1] * iL, vL = L[2] * iL, wL = L[3] * iL;
  const T uR = R[1] * iR, vR = R[2] * iR, wR = R[3] * iR;
  const T pL = g.gm1 * (L[4] - T(0.5) * (L[1] * uL + L[2] * vL + L[3] * wL));
  const T pR = g.gm1 * (R[4] - T(0.5) * (R[1] * uR + R[2] * vR + R[3] * wR));
  const T cL = Fp<T>::sqrt(g.gamma * pL * iL);
  const T cR = Fp<T>::sqrt(g.gamma * pR * iR);
  T sL = T(0), sR = T(0), iw = T(0), ua = T(0), va = T(0), wa = T(0), HL = T(0), HR = T(0), ca = T(0);
  T SL, SR;
  bool sl_first, sr_first;
  if (ws == 1) {
    const T a1 = uL - cL, b1 = uR - cR, a2 = uL + cL, b2 = uR + cR;
    sl_first = !(b1 < a1);
    sr_first = !(b2 > a2);
    SL = sl_first ? a1 : b1;
    SR = sr_first ? a2 : b2;
  } else {
    sL = Fp<T>::sqrt(L[0]);
    sR = Fp<T>::sqrt(R[0]);
    iw = Fp<T>::rcp(sL + sR);
    ua = (sL * uL + sR * uR) * iw;
    va = (sL * vL + sR * vR) * iw;
    wa = (sL * wL + sR * wR) * iw;
    HL = (L[4] + pL) * iL;
    HR = (R[4] + pR) * iR;
    const T Ha = (sL * HL + sR * HR) * iw;
    ca = Fp<T>::sqrt(g.gm1 * (Ha - T(0.5) * (ua * ua + va * va + wa * wa)));
    const T a1 = uL - cL, b1 = ua - ca, a2 = uR + cR, b2 = ua + ca;
    sl_first = !(b1 < a1);
    sr_first = !(b2 > a2);
    SL = sl_first ? a1 : b1;
    SR = sr_first ? a2 : b2;
  }
  const T aL = SL - uL;
  const T aR = SR - uR;
  const T num = pR - pL + L[0] * uL * aL - R[0] * uR * aR;
  const T den = L[0] * aL - R[0] * aR;
  const T Ss = Fp<T>::div(num, den);

  // ---- reverse: the flux of the side that enters it
  const bool left = SL >= T(0) || Ss >= T(0);
  const bool star = left ? !(SL >= T(0)) : SR > T(0);
  const T r = left ? L[0] : R[0], u = left ? uL : uR, p = left ? pL : pR;
  const T mn = left ? L[1] : R[1], m1 = left ? L[2] : R[2], m2 = left ? L[3] : R[3];
  const T E = left ? L[4] : R[4];
  const T Sk = left ? SL : SR, ak = left ? aL : aR;
  const T S = star ? Sk : T(0), a = star ? ak : T(1), Sx = star ? Ss : T(0);
  const T Dn = star ? Sk - Ss : T(1);
  const T iD = Fp<T>::rcp(Dn);
  const T rr = Fp<T>::div(a, Dn);
  const T ia = Fp<T>::rcp(a);
  const T Q = r * Sx + p * ia;
  const T G = E + (Sx - u) * Q;
  const T Us4 = rr * G;
  // F0 = mn + S (rr r - r), F1 = mn u + p + S (rr r Ss - mn), F2 = m1 u + S (rr m1 - m1),
  // F3 = m2 u + S (rr m2 - m2), F4 = (E + p) u + S (rr G - E)
  const T gS = gF[0] * (rr * r - r) + gF[1] * (rr * r * Sx - mn) + gF[2] * (rr * m1 - m1) + gF[3] * (rr * m2 - m2) +
               gF[4] * (Us4 - E);
  const T grr = S * (gF[0] * r + gF[1] * r * Sx + gF[2] * m1 + gF[3] * m2 + gF[4] * G);
  const T gG = star ? S * rr * gF[4] : T(0);
  T gr = gF[0] * S * (rr - T(1)) + gF[1] * S * rr * Sx + gG * (Sx - u) * Sx;
  T gSs_s = gF[1] * S * rr * r + gG * (Q + (Sx - u) * r);
  const T gmn = gF[0] + gF[1] * (u - S);
  T gu = gF[1] * mn + gF[2] * m1 + gF[3] * m2 + gF[4] * (E + p) - gG * Q;
  const T gp = gF[1] + gF[4] * u + gG * (Sx - u) * ia;
  T ga = -gG * (Sx - u) * p * ia * ia;
  const T gm1 = gF[2] * (u + S * (rr - T(1)));
  const T gm2 = gF[3] * (u + S * (rr - T(1)));
  const T gE = gF[4] * (u - S) + gG;
  // rr = a / (S - Ss)
  ga = ga + grr * iD;
  const T gDn = -grr * rr * iD;
  T gSk = gS + gDn;
  gSs_s = gSs_s - gDn;
  // a = S - u
  gSk = gSk + ga;
  gu = star ? gu - ga : gu;
  gr = star ? gr : T(0);
  gSk = star ? gSk : T(0);
  const T gSs = star ? gSs_s : T(0);
  T grL = left ? gr : T(0), grR = left ? T(0) : gr;
  T guL = left ? gu : T(0), guR = left ? T(0) : gu;
  T gpL = left ? gp : T(0), gpR = left ? T(0) : gp;
  T gmnL = left ? gmn : T(0), gmnR = left ? T(0) : gmn;
  T gm1L = left ? gm1 : T(0), gm1R = left ? T(0) : gm1;
  T gm2L = left ? gm2 : T(0), gm2R = left ? T(0) : gm2;
  T gEL = left ? gE : T(0), gER = left ? T(0) : gE;
  T gSL = left ? gSk : T(0), gSR = left ? T(0) : gSk;

  // S* = num / den
  const T iden = Fp<T>::rcp(den);
  const T gnum = gSs * iden;
  const T gden = -gSs * Ss * iden;
  gpR = gpR + gnum;
  gpL = gpL - gnum;
  grL = grL + gnum * uL * aL + gden * aL;
  guL = guL + gnum * L[0] * aL;
  const T gaL = T(0) + gnum * L[0] * uL + gden * L[0];
  grR = grR - gnum * uR * aR - gden * aR;
  guR = guR - gnum * R[0] * aR;
  const T gaR = T(0) - gnum * R[0] * uR - gden * R[0];
  // aL = SL - uL, aR = SR - uR
  gSL = gSL + gaL;
  guL = guL - gaL;
  gSR = gSR + gaR;
  guR = guR - gaR;

  // wave speeds
  T gcL = T(0), gcR = T(0);
  if (ws == 1) {
    guL = sl_first ? guL + gSL : guL;
    gcL = sl_first ? gcL - gSL : gcL;
    guR = sl_first ? guR : guR + gSL;
    gcR = sl_first ? gcR : gcR - gSL;
    guL = sr_first ? guL + gSR : guL;
    gcL = sr_first ? gcL + gSR : gcL;
    guR = sr_first ? guR : guR + gSR;
    gcR = sr_first ? gcR : gcR + gSR;
  } else {
    guL = sl_first ? guL + gSL : guL;
    gcL = sl_first ? -gSL : T(0);
    T gua = sl_first ? T(0) : gSL;
    T gca = sl_first ? T(0) : -gSL;
    guR = sr_first ? guR + gSR : guR;
    gcR = sr_first ? gSR : T(0);
    gua = sr_first ? gua : gua + gSR;
    gca = sr_first ? gca : gca + gSR;
    // ca = sqrt(gm1 (Ha - |ua|^2/2))
    const T gca2 = gca * T(0.5) * Fp<T>::rcp(ca);
    const T gHa = g.gm1 * gca2;
    gua = gua - g.gm1 * gca2 * ua;
    const T gva = -g.gm1 * gca2 * va;
    const T gwa = -g.gm1 * gca2 * wa;
    // Roe averages: X = (sL xL + sR xR) iw for x in u, v, w, H
    T gsL = (gua * uL + gva * vL + gwa * wL + gHa * HL) * iw;
    T gsR = (gua * uR + gva * vR + gwa * wR + gHa * HR) * iw;
    guL = guL + gua * sL * iw;
    guR = guR + gua * sR * iw;
    const T gvL = gva * sL * iw, gvR = gva * sR * iw;
    const T gwL = gwa * sL * iw, gwR = gwa * sR * iw;
    const T gHL = gHa * sL * iw, gHR = gHa * sR * iw;
    const T giw = gua * (sL * uL + sR * uR) + gva * (sL * vL + sR * vR) +
                  gwa * (sL * wL + sR * wR) + gHa * (sL * HL + sR * HR);
    const T gsum = -giw * iw * iw;
    gsL = gsL + gsum;
    gsR = gsR + gsum;
    // H = (E + p) / rho
    gEL = gEL + gHL * iL;
    gpL = gpL + gHL * iL;
    grL = grL - gHL * HL * iL;
    gER = gER + gHR * iR;
    gpR = gpR + gHR * iR;
    grR = grR - gHR * HR * iR;
    // v, w of each side through m_t / rho
    gm1L = gm1L + gvL * iL;
    gm2L = gm2L + gwL * iL;
    grL = grL - (gvL * vL + gwL * wL) * iL;
    gm1R = gm1R + gvR * iR;
    gm2R = gm2R + gwR * iR;
    grR = grR - (gvR * vR + gwR * wR) * iR;
    // sqrt(rho)
    grL = grL + gsL * T(0.5) * Fp<T>::rcp(sL);
    grR = grR + gsR * T(0.5) * Fp<T>::rcp(sR);
  }
  // c = sqrt(gamma p / rho)
  const T gxL = gcL * T(0.5) * Fp<T>::rcp(cL);
  gpL = gpL + gxL * g.gamma * iL;
  grL = grL - gxL * g.gamma * pL * iL * iL;
  const T gxR = gcR * T(0.5) * Fp<T>::rcp(cR);
  gpR = gpR + gxR * g.gamma * iR;
  grR = grR - gxR * g.gamma * pR * iR * iR;
  // p = gm1 (E - (mn u + m1 v + m2 w)/2) written on conserved variables:
  // dp/dE = gm1, dp/dm_i = -gm1 u_i, dp/drho = gm1 |u|^2 / 2
  gEL = gEL + g.gm1 * gpL;
  gmnL = gmnL - g.gm1 * gpL * uL;
  gm1L = gm1L - g.gm1 * gpL * vL;
  gm2L = gm2L - g.gm1 * gpL * wL;
  grL = grL + T(0.5) * g.gm1 * gpL * (uL * uL + vL * vL + wL * wL);
  gER = gER + g.gm1 * gpR;
  gmnR = gmnR - g.gm1 * gpR * uR;
  gm1R = gm1R - g.gm1 * gpR * vR;
  gm2R = gm2R - g.gm1 * gpR * wR;
  grR = grR + T(0.5) * g.gm1 * gpR * (uR * uR + vR * vR + wR * wR);
  // u = mn / rho
  gmnL = gmnL + guL * iL;
  grL = grL - guL * uL * iL;
  gmnR = gmnR + guR * iR;
  grR = grR - guR * uR * iR;
  gLx[0] = grL, gLx[n] = gmnL, gLx[t1] = gm1L, gLx[t2] = gm2L, gLx[4] = gEL;
  gRx[0] = grR, gRx[n] = gmnR, gRx[t1] = gm1R, gRx[t2] = gm2R, gRx[4] = gER;
}

}  // namespace gh
