// Reverse mode of the difference forms of hweno_device.h (hweno_point_diff,
// hweno_cell_diff and what they are made of), as the adjoint kernels use it:
// they are bound by the number of instructions like the stage kernels, so the
// reverse carries the scaled derivatives and the stencil differences too, and
// goes through as few intermediate quantities as the algebra allows. The
// term-by-term reverse of the direct forms is in hweno_adjoint.h, against which
// these are checked.
#pragma once

#include <type_traits>

#include "hweno_adjoint.h"
#include "hweno_device.h"

namespace hweno {

// The value x, of unknown origin to the compiler: what is computed from it is
// not taken from an earlier evaluation on the same data.
template <typename T>
HWENO_HD T anew(T x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return x;
}

// The sign of x, 0 at 0 (values of magnitude below 2^-1000 excepted).
HWENO_HD double sign_clamped(double x) { return fmin(fmax(x * 0x1p1000, -1.0), 1.0); }

// ---------------------------------------------------------------- HWENO point
// Reverse of hweno_point_diff: from the cotangents gR, gL, gT of (dR, dL, vt)
// those of its four inputs, and the forward values themselves (the basis
// cotangent needs them). MASK: which outputs take part (1 dR, 2 dL, 4 vt).
// The outputs do not change when the o_l get a common factor, so their
// cotangents are taken with P = q0 q1 q2 held: o_l = P (1 + tau / q_l) gives
//   g(tau) = sum_l P go_l / q_l,  g(q_l) = -P go_l tau / q_l^2.
// 71 instructions behind the forward's 51.
constexpr int kOutR = 1, kOutL = 2, kOutT = 4, kOutAll = 7;
template <int MASK, typename T>
HWENO_HD void hweno_point_diff_vjp(T e1_, T e2_, T S_, T D_, const PointK& k, T gR, T gL, T gT,
                                   T& dR, T& dL, T& vt, T& ge1, T& ge2, T& gS, T& gD) {
  const double e1 = (double)e1_, e2 = (double)e2_, S = (double)S_, D = (double)D_;
  constexpr double lam = Carried<T>::lam;
  constexpr double aS = 299.0 / 339.0 / lam, bD = 263845.0 / 533206.0 / lam, mD = 3.0 / 14.0 / lam;
  constexpr double kS = 71.0 / 339.0 / (lam * lam), kU = 3729.0 / 1280.0, kW = 266603.0 / 1680.0;
  constexpr double kD = 1421461.0 / 5332060.0 / (lam * lam);
  // ---- forward
  const double c = e1 + e2, s = e2 - e1;
  const double u = fma(-aS, S, c);
  const double w = fma(bD, D, s);
  double qS;
  if constexpr (lam == 1.0) qS = fma(kS * S, S, k.eps);
  else qS = fma(S, S, k.eps);
  const double q0 = fma(kW * w, w, fma(kU * u, u, fma(kD * D, D, qS)));
  const double q1 = fma(e1, e1, k.eps), q2 = fma(e2, e2, k.eps);
  const double d1 = q0 - q1, d2 = q0 - q2;
  const double ts = fabs(d1) + fabs(d2);
  const double tau = (0.25 * ts) * ts;
  const double A = q1 * q2, B = q0 * q2, C = q0 * q1;
  const double P = A * q0;
  const double o0 = fma(A, tau, P), o1 = fma(B, tau, P), o2 = fma(C, tau, P);
  const double o12 = o1 + o2;
  const double Sg = fma(k.rho, o12, o0), Sd = fma(k.rhod, o12, o0);
  const double inv = rcp_nr(Sg * Sd);
  const double iSg = Sd * inv, iSd = Sg * inv;
  const double X = fma(o1, e1, o2 * e2);
  const double base = fma(k.K, c, k.Ks * S);
  const double mm = fma(mD, D, s);
  const double om = o0 * mm;
  const double N = fma(k.X, X, o0 * base);
  double At;
  if constexpr (sizeof(T) == 8) At = fma(k.At, S, c);
  else At = fma(k.At, S, k.Ac * c);
  // ---- reverse: the numerators and normalisations
  double gN = 0.0, gm = 0.0, gSg = 0.0, nT = 0.0, gSd = 0.0;
  if constexpr ((MASK & kOutR) != 0) {
    const double d = fma(k.m, om, N) * iSg, n = (double)gR * iSg;
    dR = (T)d;
    gN = n;
    gm = n;
    gSg = -n * d;
  }
  if constexpr ((MASK & kOutL) != 0) {
    const double d = fma(-k.m, om, N) * iSg, n = (double)gL * iSg;
    dL = (T)d;
    if constexpr ((MASK & kOutR) != 0) {
      gN += n;
      gm -= n;
      gSg = fma(-n, d, gSg);
    } else {
      gN = n;
      gm = -n;
      gSg = -n * d;
    }
  }
  if constexpr ((MASK & kOutT) != 0) {
    const double v = fma(o0, At, k.Xt * X) * iSd;
    vt = (T)v;
    nT = (double)gT * iSd;
    gSd = -nT * v;
  }
  constexpr bool F = (MASK & (kOutR | kOutL)) != 0, M = (MASK & kOutT) != 0;
  if constexpr (F) gm *= k.m;
  // ---- the o_l
  double gX, go0, g12;
  if constexpr (F && M) {
    gX = fma(k.X, gN, k.Xt * nT);
    go0 = fma(gN, base, fma(gm, mm, fma(nT, At, gSg + gSd)));
    g12 = fma(k.rho, gSg, k.rhod * gSd);
  } else if constexpr (F) {
    gX = k.X * gN;
    go0 = fma(gN, base, fma(gm, mm, gSg));
    g12 = k.rho * gSg;
  } else {
    gX = k.Xt * nT;
    go0 = fma(nT, At, gSd);
    g12 = k.rhod * gSd;
  }
  const double h0 = go0 * A, h1 = fma(gX, e1, g12) * B, h2 = fma(gX, e2, g12) * C;
  // ---- tau and the q_l (cotangents z_l of q_l twice)
  const double gtau = h0 + (h1 + h2);
  const double ht = (-2.0 * tau) * rcp_nr(P);
  const double gts = ts * gtau;
  const double s1 = sign_clamped(d1), s2 = sign_clamped(d2);
  const double z0 = fma(gts, s1 + s2, (h0 * A) * ht);
  const double z1 = fma(-gts, s1, (h1 * B) * ht);
  const double z2 = fma(-gts, s2, (h2 * C) * ht);
  // ---- the inputs
  const double gu = (kU * z0) * u, gw = (kW * z0) * w;
  double gc = gu, gs = gw, rS, rD;
  if constexpr (lam == 1.0) rS = (kS * z0) * S;
  else rS = z0 * S;
  rS = fma(-aS, gu, rS);
  rD = fma(kD * z0, D, bD * gw);
  if constexpr (F) {
    const double gb = o0 * gN, gmm = o0 * gm;
    gc = fma(k.K, gb, gc);
    rS = fma(k.Ks, gb, rS);
    gs += gmm;
    rD = fma(mD, gmm, rD);
  }
  if constexpr (M) {
    const double gA = o0 * nT;
    if constexpr (sizeof(T) == 8) gc += gA;
    else gc = fma(k.Ac, gA, gc);
    rS = fma(k.At, gA, rS);
  }
  ge1 = (T)fma(gX, o1, fma(e1, z1, gc - gs));
  ge2 = (T)fma(gX, o2, fma(e2, z2, gc + gs));
  gS = (T)rS;
  gD = (T)rD;
}

// Reverse of face_derivs_diff: cotangents gR, gL of (vR, vL) -> those of the
// differences.
template <typename T>
HWENO_HD void face_derivs_diff_vjp(T gR, T gL, T& g1, T& g2, T& gS, T& gD) {
  if constexpr (sizeof(T) == 8) {
    g1 = fma(T(21.0 * kLam), gL, T(-3.0 * kLam) * gR);
    g2 = fma(T(21.0 * kLam), gR, T(-3.0 * kLam) * gL);
    gS = -(gR + gL);
    gD = T(2) * (gR - gL);
  } else {
    g1 = fma(T(1.3125), gL, T(-0.1875) * gR);
    g2 = fma(T(1.3125), gR, T(-0.1875) * gL);
    gS = T(-0.0625) * (gR + gL);
    gD = T(0.125) * (gR - gL);
  }
}

// ------------------------------------------------------------- Euler
// Cotangents of what a state's fluxes and characteristic basis are made of:
// u, v, k = |vel|^2/2, P, H = (E+P)/rho and the sound speed c. Every function
// below is written through these (rho u du = m u - ..., u (E+P) = m H), so that
// one prim_vjp serves all uses of a state.
template <typename T>
struct StateBar {
  T mu = T(0), nu = T(0), k = T(0), p = T(0), H = T(0), c = T(0);
};
// (NoBar, hweno_adjoint.h, for the scalar systems)
template <class Sys, typename T> struct StateBarOf { using type = NoBar<T>; };
template <int DIM, typename T> struct StateBarOf<Euler<DIM>, T> { using type = StateBar<T>; };

// u = m ir, v = n ir, k = (u^2+v^2)/2, P = (g-1)(E - rho k), H = (E+P) ir and,
// CHAR, c = (g P ir)^(1/2) with ich = 1/(2c)
template <bool CHAR, int DIM, typename T>
HWENO_HD void state_vjp(const Euler<DIM>& sy, const T (&U)[DIM + 2],
                        const typename Euler<DIM>::template Prim<T>& q, T H, T c, T ich,
                        StateBar<T> b, T (&gU)[DIM + 2]) {
  constexpr int E = DIM + 1;
  const T gE = q.ir * b.H;               // of E + P through H
  T gp = b.p + gE;
  if constexpr (CHAR) gp = fma(T(sy.gas) * q.ir * ich, b.c, gp);
  const T pt = T(sy.gas - 1.0) * gp;
  gU[E] += gE + pt;
  const T gk = fma(-U[0], pt, b.k);
  const T gmu = fma(q.mu, gk, b.mu);
  T x = fma(q.mu, gmu, H * b.H);
  gU[1] = fma(q.ir, gmu, gU[1]);
  if constexpr (DIM == 2) {
    const T gnu = fma(q.nu, gk, b.nu);
    x = fma(q.nu, gnu, x);
    gU[2] = fma(q.ir, gnu, gU[2]);
  }
  if constexpr (CHAR) x = fma(T(0.5) * c, b.c, x);
  gU[0] = fma(-q.ir, x, fma(-q.k, pt, gU[0]));
}
template <int DIM, typename T>
HWENO_HD void prim_vjp(const Euler<DIM>& sy, const T (&U)[DIM + 2],
                       const typename Euler<DIM>::template Prim<T>& q, StateBar<T>& b,
                       T (&gU)[DIM + 2]) {
  state_vjp<false>(sy, U, q, q.Ep * q.ir, T(0), T(0), b, gU);
}

template <int D, int DIM, typename T>
HWENO_HD void flux_vjp(const Euler<DIM>&, const T (&U)[DIM + 2],
                       const typename Euler<DIM>::template Prim<T>& q, const T (&gF)[DIM + 2],
                       StateBar<T>& b, T (&gU)[DIM + 2]) {
  const T H = q.Ep * q.ir;
  if constexpr (DIM == 1) {
    // F = (m, m u + P, m H)
    gU[1] += fma(q.mu, gF[1], fma(H, gF[2], gF[0]));
    b.mu = fma(U[1], gF[1], b.mu);
    b.H = fma(U[1], gF[2], b.H);
    b.p += gF[1];
  } else if constexpr (D == 0) {
    // F = (m, m u + P, m v, m H)
    gU[1] += fma(q.mu, gF[1], fma(q.nu, gF[2], fma(H, gF[3], gF[0])));
    b.mu = fma(U[1], gF[1], b.mu);
    b.nu = fma(U[1], gF[2], b.nu);
    b.H = fma(U[1], gF[3], b.H);
    b.p += gF[1];
  } else {
    // G = (n, n u, n v + P, n H)
    gU[2] += fma(q.mu, gF[1], fma(q.nu, gF[2], fma(H, gF[3], gF[0])));
    b.mu = fma(U[2], gF[1], b.mu);
    b.nu = fma(U[2], gF[2], b.nu);
    b.H = fma(U[2], gF[3], b.H);
    b.p += gF[2];
  }
}

// Reverse of Euler::jac (A(U) V), cotangent gO, with a = V1 - u V0 = rho du,
// b = V2 - v V0 = rho dv, dP = (g-1)(V_E - u V1 - v V2 + k V0):
// x: O = (V1, u (V1 + a) + dP, v V1 + u b, a H + u (V_E + dP)), y alike.
template <int D, int DIM, typename T>
HWENO_HD void jac_vjp(const Euler<DIM>& sy, const T (&)[DIM + 2],
                      const typename Euler<DIM>::template Prim<T>& q, const T (&V)[DIM + 2],
                      const T (&gO)[DIM + 2], StateBar<T>& s, T (&)[DIM + 2], T (&gV)[DIM + 2]) {
  constexpr int E = DIM + 1;
  const T gm1 = T(sy.gas - 1.0);
  const T H = q.Ep * q.ir;
  const T a = fma(-q.mu, V[0], V[1]);
  if constexpr (DIM == 1) {
    const T dP = gm1 * fma(q.k, V[0], fma(-q.mu, V[1], V[2]));
    const T ga = fma(q.mu, gO[1], H * gO[2]);
    const T r = q.mu * gO[2];
    const T t = gm1 * (gO[1] + r);
    gV[2] += r + t;
    gV[1] += fma(q.mu, gO[1] - t, gO[0] + ga);
    gV[0] = fma(q.k, t, fma(-q.mu, ga, gV[0]));
    s.mu = fma(V[1] + a, gO[1], fma(V[2] + dP, gO[2], fma(-V[1], t, fma(-V[0], ga, s.mu))));
    s.k = fma(V[0], t, s.k);
    s.H = fma(a, gO[2], s.H);
  } else {
    const T b = fma(-q.nu, V[0], V[2]);
    const T dP = gm1 * fma(q.k, V[0], fma(-q.nu, V[2], fma(-q.mu, V[1], V[3])));
    T ga, gb, r, t;
    if constexpr (D == 0) {
      ga = fma(q.mu, gO[1], H * gO[3]);
      gb = q.mu * gO[2];
      r = q.mu * gO[3];
      t = gm1 * (gO[1] + r);
      gV[1] += fma(q.nu, gO[2], fma(q.mu, gO[1] - t, gO[0] + ga));
      gV[2] += fma(-q.nu, t, gb);
      s.mu = fma(V[1] + a, gO[1], fma(b, gO[2], fma(V[3] + dP, gO[3], s.mu)));
      s.nu = fma(V[1], gO[2], s.nu);
      s.H = fma(a, gO[3], s.H);
    } else {
      // O = (V2, u V2 + v a, v (V2 + b) + dP, b H + v (V_E + dP))
      ga = q.nu * gO[1];
      gb = fma(q.nu, gO[2], H * gO[3]);
      r = q.nu * gO[3];
      t = gm1 * (gO[2] + r);
      gV[2] += fma(q.mu, gO[1], fma(q.nu, gO[2] - t, gO[0] + gb));
      gV[1] += fma(-q.mu, t, ga);
      s.nu = fma(V[2] + b, gO[2], fma(a, gO[1], fma(V[3] + dP, gO[3], s.nu)));
      s.mu = fma(V[2], gO[1], s.mu);
      s.H = fma(b, gO[3], s.H);
    }
    s.mu = fma(-V[1], t, fma(-V[0], ga, s.mu));
    s.nu = fma(-V[2], t, fma(-V[0], gb, s.nu));
    s.k = fma(V[0], t, s.k);
    gV[E] += r + t;
    gV[0] = fma(q.k, t, fma(-q.mu, ga, fma(-q.nu, gb, gV[0])));
  }
}

// ------------------------------------------------- characteristic basis
// Cotangent of the basis (u, v, k, c, H) through R: for a pair (x, g) of a
// back-projection U = R x and the cotangent g of U the products below are
// added; basis_bar turns the sums into the cotangent. A projection w = L U with
// cotangent gw enters as the pair (w, -L^T gw), since dL = -L dR L: the entries
// of L need no cotangent of their own.
template <typename T>
struct BasisSum {
  T mu = T(0), nu = T(0), c = T(0), t = T(0), H = T(0), k = T(0);
};
// SUB: the pair enters with the opposite sign. s0 = U_0.
template <int D, bool SUB, int N, typename T>
HWENO_HD void basis_pair(const T (&x)[N], T s0, const T (&g)[N], BasisSum<T>& b) {
  constexpr int E = N - 1;
  const T sg = SUB ? T(-1) : T(1);
  const T a = x[0] + x[E], dd = SUB ? x[0] - x[E] : x[E] - x[0];
  const T s = sg * s0;
  b.H = fma(sg * a, g[E], b.H);
  b.k = fma(sg * x[1], g[E], b.k);
  b.t = fma(dd, g[E], b.t);
  if constexpr (N == 3) {
    b.mu = fma(s, g[1], b.mu);
    b.c = fma(dd, g[1], b.c);
  } else if constexpr (D == 0) {
    b.mu = fma(s, g[1], b.mu);
    b.nu = fma(s, g[2], fma(sg * x[2], g[3], b.nu));
    b.c = fma(dd, g[1], b.c);
  } else {
    b.mu = fma(s, g[1], fma(sg * x[2], g[3], b.mu));
    b.nu = fma(s, g[2], b.nu);
    b.c = fma(dd, g[2], b.c);
  }
}
// The cotangents of u, v, k, c, H (added to those of a state).
template <int D, class Eig, typename T>
HWENO_HD void basis_bar(const Eig& e, const BasisSum<T>& b, StateBar<T>& s) {
  if constexpr (D == 0) {
    s.mu += fma(e.c, b.t, b.mu);
    s.nu += b.nu;
    s.c += fma(e.q.mu, b.t, b.c);
  } else {
    s.mu += b.mu;
    s.nu += fma(e.c, b.t, b.nu);
    s.c += fma(e.q.nu, b.t, b.c);
  }
  s.H += b.H;
  s.k += b.k;
}
// gx = R^T g
template <int D, class Eig, int N, typename T>
HWENO_HD void unproject_transposed(const Eig& e, const T (&g)[N], T (&gx)[N]) {
  if constexpr (N == 3) {
    const T gS = fma(e.q.mu, g[1], g[0]);
    const T gd = e.c * fma(e.q.mu, g[2], g[1]);
    const T ga = fma(e.H, g[2], gS);
    gx[0] = ga - gd;
    gx[1] = fma(e.q.k, g[2], gS);
    gx[2] = ga + gd;
  } else {
    const T gS = fma(e.q.mu, g[1], fma(e.q.nu, g[2], g[0]));
    const T gd = D == 0 ? e.c * fma(e.q.mu, g[3], g[1]) : e.c * fma(e.q.nu, g[3], g[2]);
    const T ga = fma(e.H, g[3], gS);
    gx[0] = ga - gd;
    gx[1] = fma(e.q.k, g[3], gS);
    gx[2] = D == 0 ? fma(e.q.nu, g[3], g[2]) : fma(e.q.mu, g[3], g[1]);
    gx[3] = ga + gd;
  }
}
// gx = L^T gw (the L of project_half)
template <int D, class Eig, int N, typename T>
HWENO_HD void project_transposed(const Eig& e, const T (&gw)[N], T (&gx)[N]) {
  constexpr int E = N - 1;
  const T gs = fma(T(-2), gw[1], gw[0] + gw[E]);
  const T pt = e.ich * (gw[0] - gw[E]);
  const T gi = -e.b1h * gs;
  gx[E] = -gi;
  if constexpr (N == 3) {
    gx[0] = fma(e.b2h, gs, fma(e.q.mu, pt, gw[1]));
    gx[1] = fma(e.q.mu, gi, -pt);
  } else if constexpr (D == 0) {
    gx[0] = fma(e.b2h, gs, fma(e.q.mu, pt, fma(-e.q.nu, gw[2], gw[1])));
    gx[1] = fma(e.q.mu, gi, -pt);
    gx[2] = fma(e.q.nu, gi, gw[2]);
  } else {
    gx[0] = fma(e.b2h, gs, fma(e.q.nu, pt, fma(-e.q.mu, gw[2], gw[1])));
    gx[1] = fma(e.q.mu, gi, gw[2]);
    gx[2] = fma(e.q.nu, gi, -pt);
  }
}

// Reverse of roe_cell_eig (the basis of Roe's matrix of UL, UR): the cotangent
// b of (u, v, k, c, H) -> contributions to both states. Forward: r = rho^-1/2,
// a = 1/(rho_L r_L + rho_R r_R), m = U_1 r, n = U_2 r, p = (g-1)(U_E - (m^2 +
// n^2)/2), X = U_E + p; mu = (m_L + m_R) a, nu = (n_L + n_R) a, H = (X_L r_L
// + X_R r_R) a, k = (mu^2 + nu^2)/2, c^2 = (g-1)(H - k).
template <int DIM, typename T>
HWENO_HD void roe_vjp(const Euler<DIM>& sy, const T (&UL)[DIM + 2], const T (&UR)[DIM + 2],
                      const typename Euler<DIM>::template CellEig<T>& e, const StateBar<T>& b,
                      T (&gUL)[DIM + 2], T (&gUR)[DIM + 2]) {
  constexpr int E = DIM + 1;
  const T gm1 = T(sy.gas - 1.0);
  const T rl = rsqrt_nr(UL[0]), rr = rsqrt_nr(UR[0]);
  const T a = rcp_nr(UL[0] * rl + UR[0] * rr);
  const T ml = UL[1] * rl, mr = UR[1] * rr;
  const T nl = DIM == 2 ? UL[2] * rl : T(0), nr = DIM == 2 ? UR[2] * rr : T(0);
  const T XL = UL[E] + gm1 * (UL[E] - T(0.5) * (ml * ml + nl * nl));
  const T XR = UR[E] + gm1 * (UR[E] - T(0.5) * (mr * mr + nr * nr));
  const T gc2 = gm1 * e.ich * b.c;
  const T gH = b.H + gc2, gk = b.k - gc2;
  const T gmu = fma(e.q.mu, gk, b.mu), gnu = fma(e.q.nu, gk, b.nu);
  const T aH = a * gH, am = a * gmu, an = a * gnu;
  // of a, over -a: shared by both states
  const T gS = -a * (fma(ml + mr, am, fma(nl + nr, an, (XL * rl + XR * rr) * aH)));
  auto side = [&](const T (&U)[DIM + 2], T r, T m, T n, T X, T (&g)[DIM + 2]) {
    const T gX = r * aH, gXp = gm1 * gX;
    const T gm = fma(-m, gXp, am);
    T gr = fma(U[1], gm, fma(X, aH, U[0] * gS));
    g[E] += gX + gXp;
    g[1] = fma(r, gm, g[1]);
    if constexpr (DIM == 2) {
      const T gn = fma(-n, gXp, an);
      gr = fma(U[2], gn, gr);
      g[2] = fma(r, gn, g[2]);
    }
    g[0] += r * fma(T(-0.5) * r * r, gr, gS);
  };
  side(UL, rl, ml, nl, XL, gUL);
  side(UR, rr, mr, nr, XR, gUR);
}

// ---------------------------------------------------- one cell's HWENO
// Reverse of the part of hweno_cell_diff that one characteristic basis e
// serves (MASK: of uR, uL, v~): the cotangents of those outputs -> added to the
// cotangents of the differences E1, E2, S, Dd; returns the basis cotangent's
// sums. (uL = U_i - R cl, so its pair enters with the opposite sign.)
template <int D, int MASK, class Sys, class Eig, typename T>
HWENO_HD void basis_cell_vjp(const Sys& sy, const PointK& k, const Eig& e, const T (&E1)[Sys::NC],
                             const T (&E2)[Sys::NC], const T (&S)[Sys::NC], const T (&Dd)[Sys::NC],
                             const T (&guR)[Sys::NC], const T (&guL)[Sys::NC],
                             const T (&gat)[Sys::NC], T (&g1)[Sys::NC], T (&g2)[Sys::NC],
                             T (&gS)[Sys::NC], T (&gD)[Sys::NC], BasisSum<T>& b) {
  constexpr int NC = Sys::NC;
  T e1[NC], e2[NC], sc[NC], dc[NC];
  sy.template project_half<D>(e, E1, e1);
  sy.template project_half<D>(e, E2, e2);
  sy.template project_half<D>(e, S, sc);
  sy.template project_half<D>(e, Dd, dc);
  T cr[NC], cl[NC], ct[NC], r[NC], l[NC], t[NC];
  if constexpr ((MASK & kOutR) != 0) unproject_transposed<D>(e, guR, r);
  if constexpr ((MASK & kOutL) != 0) unproject_transposed<D>(e, guL, l);
  if constexpr ((MASK & kOutT) != 0) unproject_transposed<D>(e, gat, t);
  T w1[NC], w2[NC], wS[NC], wD[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    // evaluated anew, not kept from the forward pass on the same cell: its
    // intermediates would not stay in the registers (y kernel 497 moves to and
    // from AGPRs an iteration and spills against 276 and none, for 224 more
    // FP64 instructions; x kernel 280 against 11)
    e1[j] = anew(e1[j]);
    e2[j] = anew(e2[j]);
    sc[j] = anew(sc[j]);
    dc[j] = anew(dc[j]);
    const T gr = (MASK & kOutR) != 0 ? r[j] : T(0), gl = (MASK & kOutL) != 0 ? -l[j] : T(0);
    const T gt = (MASK & kOutT) != 0 ? t[j] : T(0);
    hweno_point_diff_vjp<MASK, T>(e1[j], e2[j], sc[j], dc[j], k, gr, gl, gt, cr[j], cl[j], ct[j],
                                  w1[j], w2[j], wS[j], wD[j]);
  }
  if constexpr ((MASK & kOutR) != 0) basis_pair<D, false>(cr, (cr[0] + cr[NC - 1]) + cr[1], guR, b);
  if constexpr ((MASK & kOutL) != 0) basis_pair<D, true>(cl, (cl[0] + cl[NC - 1]) + cl[1], guL, b);
  if constexpr ((MASK & kOutT) != 0) basis_pair<D, false>(ct, (ct[0] + ct[NC - 1]) + ct[1], gat, b);
  auto in = [&](const T (&w)[NC], const T (&x)[NC], const T (&X)[NC], T (&g)[NC]) {
    T gx[NC];
    project_transposed<D>(e, w, gx);
    basis_pair<D, true>(x, X[0], gx, b);
#pragma unroll
    for (int c = 0; c < NC; ++c) g[c] += gx[c];
  };
  in(w1, e1, E1, g1);
  in(w2, e2, E2, g2);
  in(wS, sc, S, gS);
  in(wD, dc, Dd, gD);
}

// Reverse of hweno_cell_diff<D>, cell basis ce of U0: cotangents (guR, guL,
// gat) of (uR, uL, v~) -> added to those of the differences; what reaches U0
// through its basis goes to the state cotangent sb.
template <int D, class Sys, typename T, class Bar>
HWENO_HD void hweno_cell_diff_vjp(const Sys& sy, const PointK& k,
                                  const typename Sys::template CellEig<T>& ce,
                                  const T (&E1)[Sys::NC], const T (&E2)[Sys::NC],
                                  const T (&S)[Sys::NC], const T (&Dd)[Sys::NC],
                                  const T (&guR)[Sys::NC], const T (&guL)[Sys::NC],
                                  const T (&gat)[Sys::NC], T (&g1)[Sys::NC], T (&g2)[Sys::NC],
                                  T (&gS)[Sys::NC], T (&gD)[Sys::NC], Bar& sb) {
  if constexpr (!Sys::kChar) {
    T r, l, t, w1, w2, wS, wD;
    hweno_point_diff_vjp<kOutAll, T>(E1[0], E2[0], S[0], Dd[0], k, guR[0], -guL[0], gat[0], r, l, t,
                                     w1, w2, wS, wD);
    g1[0] += w1;
    g2[0] += w2;
    gS[0] += wS;
    gD[0] += wD;
  } else {
    BasisSum<T> b;
    basis_cell_vjp<D, kOutAll>(sy, k, ce, E1, E2, S, Dd, guR, guL, gat, g1, g2, gS, gD, b);
    basis_bar<D>(ce, b, sb);
  }
}

// The same for hweno_cell_diff_iface (the interface-basis switch): the
// right-face value in the basis of Roe's matrix of (U0, Up), the left-face
// value in that of (Um, U0), v~ in the cell basis; each application is reversed
// with its basis, whose cotangent goes to the states that define it (gUm, gU0,
// gUp). The scheduler must not interleave the three (their working sets would
// spill).
template <int D, class Sys, typename T, class Bar>
HWENO_HD void hweno_cell_diff_iface_vjp(
    const Sys& sy, const PointK& k, const typename Sys::template CellEig<T>& ce,
    const T (&Um)[Sys::NC], const T (&U0)[Sys::NC], const T (&Up)[Sys::NC], const T (&E1)[Sys::NC],
    const T (&E2)[Sys::NC], const T (&S)[Sys::NC], const T (&Dd)[Sys::NC], const T (&guR)[Sys::NC],
    const T (&guL)[Sys::NC], const T (&gat)[Sys::NC], T (&g1)[Sys::NC], T (&g2)[Sys::NC],
    T (&gS)[Sys::NC], T (&gD)[Sys::NC], T (&gUm)[Sys::NC], T (&gU0)[Sys::NC], T (&gUp)[Sys::NC],
    Bar& sb) {
  auto roe = [&](auto mask, const T (&UL)[Sys::NC], const T (&UR)[Sys::NC], T (&gl)[Sys::NC],
                 T (&gr)[Sys::NC]) {
    const auto e = sy.roe_cell_eig(UL, UR);
    BasisSum<T> b;
    basis_cell_vjp<D, decltype(mask)::value>(sy, k, e, E1, E2, S, Dd, guR, guL, gat, g1, g2, gS, gD, b);
    Bar rb{};
    basis_bar<D>(e, b, rb);
    roe_vjp(sy, UL, UR, e, rb, gl, gr);
  };
  roe(std::integral_constant<int, kOutR>{}, U0, Up, gU0, gUp);
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
  roe(std::integral_constant<int, kOutL>{}, Um, U0, gUm, gU0);
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
  BasisSum<T> b;
  basis_cell_vjp<D, kOutT>(sy, k, ce, E1, E2, S, Dd, guR, guL, gat, g1, g2, gS, gD, b);
  basis_bar<D>(ce, b, sb);
}

// The cotangent of what U0's own basis and fluxes received -> gU0.
template <class Sys, typename T, class Bar>
HWENO_HD void cell_state_vjp(const Sys& sy, const T (&U0)[Sys::NC],
                             const typename Sys::template CellEig<T>& ce, const Bar& sb,
                             T (&gU0)[Sys::NC]) {
  if constexpr (Sys::kChar) state_vjp<true>(sy, U0, ce.q, ce.H, ce.c, ce.ich, sb, gU0);
}

}  // namespace hweno
