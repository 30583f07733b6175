// Vector-Jacobian product of the HLLD flux (mhd_hlld.h): the cotangents of both
// states of a face from the cotangent of its flux, one reverse sweep instead of
// one forward-mode (dual number) solve per state component.
#pragma once

#include <hip/hip_runtime.h>

#include "dg_math.h"
#include "dual.h"
#include "mhd_hlld.h"

namespace dg {

// The same product in forward mode: one dual-number solve per state component.
template <typename T, int D>
__device__ __forceinline__ void hlld_vjp_forward(const T* uL, const T* uR, T gamma, T eps,
                                                 const T* Fb, T* ubL, T* ubR) {
#pragma unroll 1
  for (int k = 0; k < 16; ++k) {
    Dual<T> dL[8], dR[8], F[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      dL[j] = Dual<T>(uL[j], T(j == k ? 1 : 0));
      dR[j] = Dual<T>(uR[j], T(j + 8 == k ? 1 : 0));
    }
    dL[5 + D].d = dR[5 + D].d = T(0.5) * (dL[5 + D].d + dR[5 + D].d);
    bool bad = false;
    hlld_axis<Dual<T>, D>(dL, dR, Dual<T>(gamma, T(0)), Dual<T>(eps, T(0)), F, bad);
    T acc = T(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc = fma(Fb[j], F[j].d, acc);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      ubL[j] = j == k ? acc : ubL[j];
      ubR[j] = j + 8 == k ? acc : ubR[j];
    }
  }
}

// uL, uR: lab-frame states in the order rho, mx, my, mz, E, Bx, By, Bz, both
// carrying the face's normal field B[D]; Fb: cotangent of the flux of
// hlld_axis<T, D> (its B[D] entry is ignored: that flux is identically zero).
// Returns ubL, ubR; the entry 5 + D of each is the cotangent of its side's own
// normal field where the face's is the average of the two (half of the total).
//
// The branch differentiated is the one hlld_axis takes, with its conventions at
// kinks: min and max take the left state on ties, a degenerate star state
// (|den| <= eps scale) keeps the outer transverse values with no derivative
// through den, the square root of a zero discriminant has derivative zero.
//
// Where a star state is nearly degenerate (|den| < 2e-4 scale in FP64) the
// Jacobian is ill-conditioned: its entries carry a relative error of about eps
// (scale / den)^2 that depends on the order of the operations.  Those faces (none
// in most flows; 1e-5 of the faces where the field dominates) take the forward
// mode, in the arithmetic of the forward flux, so that they do not depend on the
// sweep's.  Elsewhere the two agree to 1e-8 at worst.  That is a matter of agreement,
// not of accuracy: against extended precision both have the same error, in FP32 too
// (400,000 random faces, median and 99th percentile within 7% of each other: den/scale
// above 0.1 1e-7 and 4e-7 of the largest entry, 1e-3..1e-2 3e-6 and 5e-5, 1e-5..1e-4
// 9e-4 and 0.14), so FP32 faces all take the sweep.
//
// The fan is symmetric under a swap of its sides, so the sweep is written once
// for the side `a` the interface lies on and the other side `o`.  In the fan the
// jump conditions make the flux of hlld_axis the flux of the region's state,
//   (r s, r s^2 + p - Bn^2, r s V - Bn B, (E + p) s - Bn V.B, B s - Bn V)
// with r, s, p, V, B, E the state outside the fan (s = u), the single-star or
// the double-star state (s = S_M), plus b (u - S_M) in the field components
// where the star state is degenerate.
template <typename T, int D>
__device__ __forceinline__ void hlld_vjp(const T* uL, const T* uR, T gamma, T eps, const T* Fb,
                                         T* ubL, T* ubR) {
  constexpr int n = D, t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const T gm1 = gamma - T(1);
  const T Bn = uL[5 + n], Bn2 = Bn * Bn;
  T r[2], ir[2], u[2], v[2], w[2], b1[2], b2[2], E[2], pm[2], pg[2], pT[2], cf[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const T* q = s == 0 ? uL : uR;
    r[s] = q[0];
    ir[s] = rcp(q[0]);
    u[s] = q[1 + n] * ir[s];
    v[s] = q[1 + t1] * ir[s];
    w[s] = q[1 + t2] * ir[s];
    b1[s] = q[5 + t1];
    b2[s] = q[5 + t2];
    E[s] = q[4];
    pm[s] = T(0.5) * (Bn2 + b1[s] * b1[s] + b2[s] * b2[s]);
    pg[s] = gm1 * (E[s] - T(0.5) * (q[1 + n] * u[s] + q[1 + t1] * v[s] + q[1 + t2] * w[s]) - pm[s]);
    pT[s] = pg[s] + pm[s];
    const T a2 = gamma * pg[s] * ir[s];
    const T sb = a2 + T(2) * pm[s] * ir[s];
    const T disc = fmax(sb * sb - T(4) * a2 * Bn2 * ir[s], T(0));
    cf[s] = sqrt_pos(T(0.5) * (sb + sqrt_nn(disc)));
  }
  const bool cR = cf[1] > cf[0];     // the side that sets max(c_f)
  const bool loR = u[1] < u[0];      // the side that sets min(u)
  const bool hiR = u[1] > u[0];      // the side that sets max(u)
  const T cmax = cR ? cf[1] : cf[0];
  const T SL = (loR ? u[1] : u[0]) - cmax;
  const T SR = (hiR ? u[1] : u[0]) + cmax;
  const T dL = (SL - u[0]) * r[0], dR = (SR - u[1]) * r[1];
  const T idn = rcp(dR - dL);
  const T SM = (dR * u[1] - dL * u[0] - pT[1] + pT[0]) * idn;
  const T du = u[1] - u[0];
  const T pTs = (dR * pT[0] - dL * pT[1] + dL * dR * du) * idn;
  // sides a (index 0) and o (index 1)
  const bool lft = SM >= T(0);
  auto swap = [lft](T* x) {
    const T x0 = lft ? x[0] : x[1], x1 = lft ? x[1] : x[0];
    x[0] = x0;
    x[1] = x1;
  };
  T S[2] = {SL, SR}, d[2] = {dL, dR};
  swap(r);
  swap(ir);
  swap(u);
  swap(v);
  swap(w);
  swap(b1);
  swap(b2);
  swap(E);
  swap(pm);
  swap(pg);
  swap(pT);
  swap(S);
  swap(d);
  bool near = false;
  const T sig = lft ? T(-1) : T(1);
  const T sgn = Bn < T(0) ? T(-1) : T(1);
  const T tau = lft ? sgn : -sgn;  // (x_R - x_L) sgn = (x_o - x_a) tau
  T iSM[2], rs[2], iden[2], fv[2], fb[2], vs[2], ws[2], c1[2], c2[2], sq[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const T SmM = S[s] - SM, Su = S[s] - u[s];
    iSM[s] = rcp(SmM);
    rs[s] = d[s] * iSM[s];
    const T den = d[s] * SmM - Bn2;
    const T scale = d[s] * Su + Bn2;
    const bool deg = fabs(den) <= eps * scale;
    if (sizeof(T) == 8) near |= !deg && fabs(den) < T(2e-4) * scale;
    iden[s] = deg ? T(0) : rcp(den);
    fv[s] = deg ? T(0) : Bn * (SM - u[s]) * iden[s];
    fb[s] = deg ? T(1) : (d[s] * Su - Bn2) * iden[s];
    vs[s] = v[s] - b1[s] * fv[s];
    ws[s] = w[s] - b2[s] * fv[s];
    c1[s] = b1[s] * fb[s];
    c2[s] = b2[s] * fb[s];
    sq[s] = sqrt_pos(rs[s]);
  }
  const T isum = rcp(sq[0] + sq[1]);
  const T dv = (vs[1] - vs[0]) * tau, dw = (ws[1] - ws[0]) * tau;
  const T vss = (sq[0] * vs[0] + sq[1] * vs[1] + (c1[1] - c1[0]) * tau) * isum;
  const T wss = (sq[0] * ws[0] + sq[1] * ws[1] + (c2[1] - c2[0]) * tau) * isum;
  const T c1ss = (sq[0] * c1[1] + sq[1] * c1[0] + sq[0] * sq[1] * dv) * isum;
  const T c2ss = (sq[0] * c2[1] + sq[1] * c2[0] + sq[0] * sq[1] * dw) * isum;
  const T isq = rcp(sq[0]);
  const T Ss = SM + sig * fabs(Bn) * isq;
  const bool outer = lft ? (SL >= T(0)) : (SR <= T(0));
  const bool single = lft ? (Ss >= T(0)) : (Ss <= T(0));
  const bool dbl = !outer && !single;
  const T vB = u[0] * Bn + v[0] * b1[0] + w[0] * b2[0];
  const T vBs = SM * Bn + vs[0] * c1[0] + ws[0] * c2[0];
  const T vBss = SM * Bn + vss * c1ss + wss * c2ss;
  const T Es = ((S[0] - u[0]) * E[0] - pT[0] * u[0] + pTs * SM + Bn * (vB - vBs)) * iSM[0];
  const T kE = sig * sgn;
  const T Ess = Es + kE * sq[0] * (vBs - vBss);
  // the region's state
  const T xr = outer ? r[0] : rs[0], xs = outer ? u[0] : SM, xp = outer ? pT[0] : pTs;
  const T xV = outer ? v[0] : (dbl ? vss : vs[0]), xW = outer ? w[0] : (dbl ? wss : ws[0]);
  const T xB = outer ? b1[0] : (dbl ? c1ss : c1[0]), xC = outer ? b2[0] : (dbl ? c2ss : c2[0]);
  const T xE = outer ? E[0] : (dbl ? Ess : Es), xvB = outer ? vB : (dbl ? vBss : vBs);

  // ---- reverse sweep: cotangents of the region's state
  const T f0 = Fb[0], f1 = Fb[1 + n], f2 = Fb[1 + t1], f3 = Fb[1 + t2], f4 = Fb[4];
  const T f5 = Fb[5 + t1], f6 = Fb[5 + t2];
  const T mom = f0 + f2 * xV + f3 * xW;
  const T xrb = xs * (mom + f1 * xs);
  T xsb = xr * (mom + T(2) * f1 * xs) + f4 * (xE + xp) + f5 * xB + f6 * xC;
  const T G = xr * xs;
  const T xpb = f1 + f4 * xs;
  T Vb = f2 * G - f5 * Bn, Wb = f3 * G - f6 * Bn;
  T Bb = f5 * xs - f2 * Bn, Cb = f6 * xs - f3 * Bn;
  const T Eb = f4 * xs;
  T vBxb = -f4 * Bn;
  T Bnb = -(T(2) * Bn * f1 + f2 * xB + f3 * xC + f4 * xvB + f5 * xV + f6 * xW);
  // primitive cotangents of the sides (a, o)
  T rb[2] = {outer ? xrb : T(0), T(0)};
  T ub[2] = {outer ? xsb : T(0), T(0)};
  T vb[2] = {outer ? Vb : T(0), T(0)};
  T wb[2] = {outer ? Wb : T(0), T(0)};
  T b1b[2] = {outer ? Bb : T(0), T(0)};
  T b2b[2] = {outer ? Cb : T(0), T(0)};
  T Ecb = outer ? Eb : T(0);  // E of side a (side o's energy enters through its pressure only)
  T pTb[2] = {outer ? xpb : T(0), T(0)};
  T vBb = outer ? vBxb : T(0);
  // from here on the fan: zero where the flux is the outer one
  const T z = outer ? T(0) : T(1);
  T SMb = z * xsb, pTsb = z * xpb;
  const bool deg0 = iden[0] == T(0);
  const T fdeg = deg0 ? z * (f5 * b1[0] + f6 * b2[0]) : T(0);  // b (u - S_M) terms
  SMb -= fdeg;
  ub[0] += fdeg;
  b1b[0] += deg0 ? z * f5 * (u[0] - SM) : T(0);
  b2b[0] += deg0 ? z * f6 * (u[0] - SM) : T(0);
  T rsb[2] = {z * xrb, T(0)};
  Vb *= z;
  Wb *= z;
  Bb *= z;
  Cb *= z;
  vBxb *= z;
  const T Esb = z * Eb;
  T Sb[2] = {T(0), T(0)}, db[2] = {T(0), T(0)};
  // double star: E** = E* + k sqrt(r*) (v*.B* - v**.B**), then v**, B**
  const T y = dbl ? T(1) : T(0);
  const T ke = y * kE * Esb;
  const T vBssb = y * vBxb - ke * sq[0];
  T vBsb = (vBxb - y * vBxb) + ke * sq[0];
  T sqb[2] = {ke * (vBs - vBss), T(0)};
  SMb = fma(vBssb, Bn, SMb);
  Bnb = fma(vBssb, SM, Bnb);
  const T A1 = (y * Vb + vBssb * c1ss) * isum, A2 = (y * Wb + vBssb * c2ss) * isum;
  const T C1 = (y * Bb + vBssb * vss) * isum, C2 = (y * Cb + vBssb * wss) * isum;
  const T x1 = C1 * sq[0] * sq[1] * tau, x2 = C2 * sq[0] * sq[1] * tau;
  T vsb[2] = {(Vb - y * Vb) + A1 * sq[0] - x1, A1 * sq[1] + x1};
  T wsb[2] = {(Wb - y * Wb) + A2 * sq[0] - x2, A2 * sq[1] + x2};
  T c1b[2] = {(Bb - y * Bb) + C1 * sq[1] - A1 * tau, C1 * sq[0] + A1 * tau};
  T c2b[2] = {(Cb - y * Cb) + C2 * sq[1] - A2 * tau, C2 * sq[0] + A2 * tau};
  sqb[0] += A1 * (vs[0] - vss) + A2 * (ws[0] - wss) + C1 * (c1[1] + sq[1] * dv - c1ss) +
            C2 * (c2[1] + sq[1] * dw - c2ss);
  sqb[1] += A1 * (vs[1] - vss) + A2 * (ws[1] - wss) + C1 * (c1[0] + sq[0] * dv - c1ss) +
            C2 * (c2[0] + sq[0] * dw - c2ss);
  rsb[0] += T(0.5) * sqb[0] * isq;
  rsb[1] += T(0.5) * sqb[1] * rcp(sq[1]);
  // E* of side a
  const T X = Esb * iSM[0];
  Sb[0] += X * (E[0] - Es);
  ub[0] -= X * (E[0] + pT[0]);
  Ecb += X * (S[0] - u[0]);
  pTb[0] -= X * u[0];
  pTsb = fma(X, SM, pTsb);
  SMb += X * (pTs + Es);
  Bnb += X * (vB - vBs);
  vBb = fma(X, Bn, vBb);
  vBsb = fma(-X, Bn, vBsb);
  // v*.B*, v.B of side a
  SMb = fma(vBsb, Bn, SMb);
  Bnb = fma(vBsb, SM, Bnb);
  vsb[0] = fma(vBsb, c1[0], vsb[0]);
  wsb[0] = fma(vBsb, c2[0], wsb[0]);
  c1b[0] = fma(vBsb, vs[0], c1b[0]);
  c2b[0] = fma(vBsb, ws[0], c2b[0]);
  ub[0] = fma(vBb, Bn, ub[0]);
  Bnb = fma(vBb, u[0], Bnb);
  vb[0] = fma(vBb, b1[0], vb[0]);
  wb[0] = fma(vBb, b2[0], wb[0]);
  b1b[0] = fma(vBb, v[0], b1b[0]);
  b2b[0] = fma(vBb, w[0], b2b[0]);
  // single-star states of both sides
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    vb[s] += vsb[s];
    wb[s] += wsb[s];
    b1b[s] += c1b[s] * fb[s] - vsb[s] * fv[s];
    b2b[s] += c2b[s] * fb[s] - wsb[s] * fv[s];
    // through 1/den (iden = 0 in a degenerate star state)
    const T fvb = -(vsb[s] * b1[s] + wsb[s] * b2[s]) * iden[s];
    const T fbb = (c1b[s] * b1[s] + c2b[s] * b2[s]) * iden[s];
    const T denb = -(fvb * fv[s] + fbb * fb[s]);
    Bnb += fvb * (SM - u[s]) - T(2) * Bn * (fbb + denb);
    const T fB = fvb * Bn, fd = fbb * d[s], dd = denb * d[s];
    SMb += fB - dd;
    ub[s] -= fB + fd;
    Sb[s] += fd + dd;
    db[s] += fbb * (S[s] - u[s]) + denb * (S[s] - SM);
    const T ri = rsb[s] * iSM[s];
    db[s] += ri;
    Sb[s] -= ri * rs[s];
    SMb = fma(ri, rs[s], SMb);
  }
  // S_M and p*_T: with the sides' order a, o both are the same expressions
  // (numerator and denominator change sign together)
  const T id = lft ? idn : -idn;  // 1/(d_o - d_a)
  const T Y = SMb * id, Z = pTsb * id;
  const T duo = u[1] - u[0];
  db[1] += Y * (u[1] - SM) + Z * (pT[0] + d[0] * duo - pTs);
  db[0] += Y * (SM - u[0]) + Z * (pTs - pT[1] + d[1] * duo);
  const T Zdd = Z * d[0] * d[1];
  ub[1] += Y * d[1] + Zdd;
  ub[0] -= Y * d[0] + Zdd;
  pTb[1] -= Y + Z * d[0];
  pTb[0] += Y + Z * d[1];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    Sb[s] = fma(db[s], r[s], Sb[s]);
    ub[s] = fma(-db[s], r[s], ub[s]);
    rb[s] = fma(db[s], S[s] - u[s], rb[s]);
  }
  // outer speeds S_L = min(u) - max(c_f), S_R = max(u) + max(c_f)
  const T SLb = lft ? Sb[0] : Sb[1], SRb = lft ? Sb[1] : Sb[0];
  const bool loO = loR == lft, hiO = hiR == lft;  // the side that sets it is o
  ub[0] += (loO ? T(0) : SLb) + (hiO ? T(0) : SRb);
  ub[1] += (loO ? SLb : T(0)) + (hiO ? SRb : T(0));
  // c_f of the side that sets the maximum
  const bool cO = cR == lft;
  const T cir = cO ? ir[1] : ir[0], cpg = cO ? pg[1] : pg[0], cpm = cO ? pm[1] : pm[0];
  const T a2 = gamma * cpg * cir;
  const T sb = a2 + T(2) * cpm * cir;
  const T disc = sb * sb - T(4) * a2 * Bn2 * cir;
  const T hq = T(0.25) * (SRb - SLb) * rcp(cmax);
  const T discb = disc > T(0) ? T(0.5) * hq * rcp(sqrt_pos(disc)) : T(0);
  const T sbb = fma(T(2) * sb, discb, hq);
  const T k4 = T(4) * discb * Bn;
  const T a2b = sbb - k4 * Bn * cir;
  Bnb -= T(2) * k4 * a2 * cir;
  const T cirb = T(2) * cpm * sbb + gamma * cpg * a2b - k4 * Bn * a2;
  const T cpgb = gamma * cir * a2b, cpmb = T(2) * cir * sbb;
  // primitive to conserved
  T ob[2][8];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const bool here = (s == 1) == cO;
    const T pgb = pTb[s] + (here ? cpgb : T(0));
    const T irb = here ? cirb : T(0);
    const T gp = gm1 * pgb;
    const T pmb = pTb[s] + (here ? cpmb : T(0)) - gp;
    const T mnb = (ub[s]) * ir[s] - gp * u[s];
    const T m1b = vb[s] * ir[s] - gp * v[s];
    const T m2b = wb[s] * ir[s] - gp * w[s];
    // d/d rho at fixed momenta: through u, v, w, 1/rho and p_g = ... - |m|^2/(2 rho)
    ob[s][0] = rb[s] - ir[s] * (ub[s] * u[s] + vb[s] * v[s] + wb[s] * w[s] + ir[s] * irb) +
               T(0.5) * gp * (u[s] * u[s] + v[s] * v[s] + w[s] * w[s]);
    ob[s][1 + n] = mnb;
    ob[s][1 + t1] = m1b;
    ob[s][1 + t2] = m2b;
    ob[s][4] = gp + (s == 0 ? Ecb : T(0));
    Bnb = fma(pmb, Bn, Bnb);
    ob[s][5 + t1] = fma(pmb, b1[s], b1b[s]);
    ob[s][5 + t2] = fma(pmb, b2[s], b2b[s]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (k == 5 + n) continue;
    ubL[k] = lft ? ob[0][k] : ob[1][k];
    ubR[k] = lft ? ob[1][k] : ob[0][k];
  }
  ubL[5 + n] = ubR[5 + n] = T(0.5) * Bnb;
  if (near) hlld_vjp_forward<T, D>(uL, uR, gamma, eps, Fb, ubL, ubR);
}

// Volume term at one point: ub (rho, mx, my, mz, E, Bx, By, Bz) is the
// cotangent of the point state u from the cotangents of its fluxes along the
// first NE axes: feb[e][v] of the hydro flux of variable v along axis e, and of
// the three independent induction fluxes, k01 of B_x v_y - v_x B_y, k02 of
// B_x v_z - v_x B_z, k12 of B_y v_z - v_y B_z.
template <typename T, int NE>
__device__ __forceinline__ void mhd_flux_vjp(const T* u, T gamma, const T (*feb)[5], T k01, T k02,
                                             T k12, T* ub) {
  const T gm1 = gamma - T(1);
  const T ir = rcp(u[0]);
  const T* B = u + 5;
  const T v[3] = {u[1] * ir, u[2] * ir, u[3] * ir};
  const T pm = T(0.5) * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
  const T pg = gm1 * (u[4] - T(0.5) * (u[1] * v[0] + u[2] * v[1] + u[3] * v[2]) - pm);
  const T Ep = u[4] + pg + pm;
  const T vB = v[0] * B[0] + v[1] * B[1] + v[2] * B[2];
  T mb[3] = {T(0), T(0), T(0)}, vb[3] = {T(0), T(0), T(0)}, Bb[3] = {T(0), T(0), T(0)};
  T pTb = T(0), vBb = T(0), Eb = T(0);
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const T f4 = feb[e][4];
    T mf = f4 * Ep, Bf = f4 * vB;
    mb[e] += feb[e][0];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const T f = feb[e][1 + k];
      mb[k] = fma(f, v[e], mb[k]);
      mf = fma(f, u[1 + k], mf);
      Bb[k] = fma(-f, B[e], Bb[k]);
      Bf = fma(f, B[k], Bf);
    }
    vb[e] += mf;
    Bb[e] -= Bf;
    pTb += feb[e][1 + e] + f4 * v[e];
    vBb = fma(-f4, B[e], vBb);
    Eb = fma(f4, v[e], Eb);
  }
  Bb[0] += k01 * v[1] + k02 * v[2];
  Bb[1] += k12 * v[2] - k01 * v[0];
  Bb[2] -= k02 * v[0] + k12 * v[1];
  vb[0] -= k01 * B[1] + k02 * B[2];
  vb[1] += k01 * B[0] - k12 * B[2];
  vb[2] += k02 * B[0] + k12 * B[1];
  const T gp = gm1 * pTb, pmb = pTb - gp;
  T s = T(0), v2 = T(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    vb[k] = fma(vBb, B[k], vb[k]);
    Bb[k] += vBb * v[k] + pmb * B[k];
    s = fma(vb[k], v[k], s);
    v2 = fma(v[k], v[k], v2);
    ub[1 + k] = mb[k] + vb[k] * ir - gp * v[k];
    ub[5 + k] = Bb[k];
  }
  ub[0] = T(0.5) * gp * v2 - s * ir;
  ub[4] = Eb + gp;
}

}  // namespace dg
