// One-dimensional building blocks of the sum-factorised stage kernels: the
// Gauss rule and the scaled Legendre polynomials as compile-time constants,
// and contractions of a total-degree polynomial one axis at a time.
#pragma once

#include "dg_device.h"

namespace dg {

constexpr double csqrt(double x) {
  double y = x > 1.0 ? x : 1.0;
  for (int i = 0; i < 60; ++i) y = 0.5 * (y + x / y);
  return y;
}

// Legendre polynomial P_n(x) and its derivative by the three-term recurrence.
constexpr double legendre_p(int n, double x) {
  double p0 = 1.0, p1 = x;
  if (n == 0) return 1.0;
  for (int j = 2; j <= n; ++j) {
    const double p2 = ((2 * j - 1) * x * p1 - (j - 1) * p0) / j;
    p0 = p1;
    p1 = p2;
  }
  return p1;
}
constexpr double legendre_d(int n, double x) {
  return n == 0 ? 0.0 : n * (x * legendre_p(n, x) - legendre_p(n - 1, x)) / (x * x - 1.0);
}

// Gauss-Legendre rule with K + 1 points (nodes ascending), P~_e = sqrt(2e+1)
// P_e at the nodes and at +1, and the expansion P~_e' = sum_j dc[e][j] P~_j
// (j = e-1, e-3, ..: P_e' = sum (2j+1) P_j).
template <int K>
struct Line {
  static constexpr int n1 = K + 1;
  double x[n1], w[n1], p[n1][n1], b[n1], dc[n1][n1];
  double ph[2][n1][n1];  // P~_e at (x_i - 1) / 2 and (x_i + 1) / 2: the nodes of the two halves
  double rh[n1][n1];     // P~_e((x + 1) / 2) = sum_j rh[e][j] P~_j(x), j <= e; the other half's: (-1)^(e + j) rh
  constexpr Line() : x(), w(), p(), b(), dc(), ph(), rh() {
    for (int i = 0; i < n1 / 2; ++i) {
      // bisection to the root i of P_{n1} in (0, 1), then Newton steps
      double lo = 0.0, hi = 1.0;
      int seen = 0;
      const int want = n1 / 2 - i;  // the want-th positive root from 0
      double prev = legendre_p(n1, 1e-3);
      for (int s = 1; s <= 1000; ++s) {
        const double xs = s * 1e-3, v = legendre_p(n1, xs);
        if (s > 1 && (prev < 0.0) != (v < 0.0)) {
          if (++seen == want) {
            lo = xs - 1e-3;
            hi = xs;
          }
        }
        prev = v;
      }
      double r = 0.5 * (lo + hi);
      for (int it = 0; it < 20; ++it) r -= legendre_p(n1, r) / legendre_d(n1, r);
      x[n1 - 1 - i] = r;
      x[i] = -r;
    }
    for (int i = 0; i < n1; ++i) {
      const double d = legendre_d(n1, x[i]);
      w[i] = 2.0 / ((1.0 - x[i] * x[i]) * d * d);
      for (int e = 0; e < n1; ++e) {
        p[i][e] = csqrt(2 * e + 1) * legendre_p(e, x[i]);
        for (int h = 0; h < 2; ++h) ph[h][i][e] = csqrt(2 * e + 1) * legendre_p(e, 0.5 * (x[i] + (h ? 1.0 : -1.0)));
      }
    }
    for (int e = 0; e < n1; ++e) {
      b[e] = csqrt(2 * e + 1);
      for (int j = 0; j < e; ++j) dc[e][j] = (e - j) % 2 ? csqrt(2 * e + 1) * csqrt(2 * j + 1) : 0.0;
      for (int j = 0; j <= e; ++j)
        for (int i = 0; i < n1; ++i) rh[e][j] += 0.5 * w[i] * ph[1][i][e] * p[i][j];
    }
  }
};

// The same numbers in constant memory, for loops over nodes that stay loops
// (uniform index: scalar loads).
__constant__ const Line<1> c_line1{};
__constant__ const Line<2> c_line2{};
__constant__ const Line<3> c_line3{};
__constant__ const Line<4> c_line4{};
template <int K>
__device__ __forceinline__ const Line<K> &line_const() {
  if constexpr (K == 1) return c_line1;
  else if constexpr (K == 2) return c_line2;
  else if constexpr (K == 3) return c_line3;
  else return c_line4;
}

// Index of the mode with exponents e of a total-degree basis in D variables
// (order of mode_exp); D = 1: the exponent itself.
template <int D>
__host__ __device__ constexpr int mode_index(int ex, int ey, int ez) {
  if (D == 1) return ex;
  const int t = ex + ey + ez;
  if (D == 2) return t * (t + 1) / 2 + ey;
  const int r = t - ex;  // among degree t: x-exponent descending, then y-exponent descending
  return t * (t + 1) * (t + 2) / 6 + r * (r + 1) / 2 + ez;
}

// values u[0..K] at the Gauss nodes of sum_{e <= M} c[e] P~_e, M <= K: the
// nodes come in pairs +-x, whose even and odd parts are formed once
template <int K, int M>
__device__ __forceinline__ void line_values(const double (&c)[M + 1], double (&u)[K + 1]) {
#pragma clang fp contract(off)
  constexpr Line<K> L{};
  constexpr int n1 = K + 1;
  if constexpr (M == 0) {
#pragma unroll
    for (int i = 0; i < n1; ++i) u[i] = c[0];
  } else if constexpr (M <= 2) {  // one odd term: two multiply-adds per pair beat the sums
#pragma unroll
    for (int i = 0; i < n1 / 2; ++i) {
      double e = c[0];
      if constexpr (M == 2) e = fma(c[2], L.p[i][2], e);
      u[i] = fma(c[1], L.p[i][1], e);
      u[K - i] = fma(c[1], L.p[K - i][1], e);
    }
    if constexpr (n1 % 2) {
      u[K / 2] = c[0];
      if constexpr (M == 2) u[K / 2] = fma(c[2], L.p[K / 2][2], c[0]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < n1 / 2; ++i) {
      double e = fma(c[2], L.p[i][2], c[0]);
      if constexpr (M >= 4) e = fma(c[4], L.p[i][4], e);
      const double o = fma(c[3], L.p[i][3], c[1] * L.p[i][1]);
      u[i] = e + o;
      u[K - i] = e - o;
    }
    if constexpr (n1 % 2) {
      u[K / 2] = fma(c[2], L.p[K / 2][2], c[0]);
      if constexpr (M >= 4) u[K / 2] = fma(c[4], L.p[K / 2][4], u[K / 2]);
    }
  }
}

// s[e] = sum_i w_i P~_e(x_i) f[i] for e <= M
template <int K, int M>
__device__ __forceinline__ void line_moments(const double (&f)[K + 1], double (&s)[M + 1]) {
  constexpr Line<K> L{};
  constexpr int n1 = K + 1, h = n1 / 2;
  double sp[h > 0 ? h : 1], sm[h > 0 ? h : 1];
#pragma unroll
  for (int i = 0; i < h; ++i) {
    sp[i] = f[K - i] + f[i];
    if constexpr (M >= 1) sm[i] = f[K - i] - f[i];
  }
#pragma unroll
  for (int e = 0; e <= M; ++e) {
    double t = 0.0;
    bool first = true;
    if (e % 2 == 0 && n1 % 2) {
      t = (L.w[K / 2] * L.p[K / 2][e]) * f[K / 2];
      first = false;
    }
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const double cw = L.w[K - i] * L.p[K - i][e], v = e % 2 ? sm[i] : sp[i];
      t = first ? cw * v : fma(cw, v, t);
      first = false;
    }
    s[e] = t;
  }
}

// reciprocal and reciprocal square root: one third-order step on the
// hardware estimates (x r = 1 - e: r (1 + e + e^2); x y^2 = 1 - e:
// y (1 + e/2 + 3 e^2 / 8)); the estimates' error is below 2^-20, so the
// neglected term is below 2^-60
__device__ __forceinline__ double rcp3(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsq3(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// HLLC flux in +A between UL and UR, wave-speed bounds as hllc.  With f the
// mass flux of the star region's side K (sel below), the flux of every
// tangential momentum is v_t f, and the normal momentum and energy fluxes
// follow from f, p_K and A = S_K rho_K (S_K - u_K) / (S_K - S*), so only
// seven quantities of the two sides are selected and the flux itself takes
// twelve operations (hllc forms U*_K and F_K first).  f = rho_K (S_K - u_K)
// S* / (S_K - S*) where 0 lies between S_K and S*, else the side's own
// momentum m_K, not rounded again (rho_K u_K instead made a cold supersonic
// disc's right-hand side 1.3 to 1.7 times as far from exact).  A trace without
// a real sound speed gives NaN in every flux as in hllc (0 (c_L + c_R) is added
// to S*: the hardware's min and max drop a NaN operand; and S* enters f with
// the factor 0 where f is m_K).
template <int D, int A, int FX>
__device__ __forceinline__ void hllc_line(const double (&UL)[D + 2], const double (&UR)[D + 2], double g, double (&F)[D + 2]) {
#pragma clang fp contract(off)
  const double gm1 = g - 1.0;
  const double rsL = rsq3(UL[0]), rsR = rsq3(UR[0]);
  const double irL = rsL * rsL, irR = rsR * rsR;
  double vL[D], vR[D], keL = 0.0, keR = 0.0;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    vL[b] = UL[1 + b] * irL;
    vR[b] = UR[1 + b] * irR;
    keL = b == 0 ? UL[1] * vL[0] : fma(UL[1 + b], vL[b], keL);
    keR = b == 0 ? UR[1] * vR[0] : fma(UR[1 + b], vR[b], keR);
  }
  const double uL = vL[A], uR = vR[A];
  const double pL = gm1 * fma(-0.5, keL, UL[D + 1]), pR = gm1 * fma(-0.5, keR, UR[D + 1]);
  const double xL = g * pL * irL, xR = g * pR * irR;
  const double cL = xL * rsq3(xL), cR = xR * rsq3(xR);
  const double eL = UL[D + 1] * irL, eR = UR[D + 1] * irR;
  double SL, SR;
  if constexpr (FX == DG_HLLC_DAVIS) {
    SL = fmin(uL - cL, uR - cR);
    SR = fmax(uL + cL, uR + cR);
  } else {
    const double sL = UL[0] * rsL, sR = UR[0] * rsR;
    const double is = rcp3(sL + sR), wL = sL * is, wR = sR * is;
    double q2 = 0.0, ut = 0.0;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const double vt = fma(wL, vL[b], wR * vR[b]);
      q2 = b == 0 ? vt * vt : fma(vt, vt, q2);
      if (b == A) ut = vt;
    }
    const double Ht = fma(wL, fma(pL, irL, eL), wR * fma(pR, irR, eR));
    // a squared Roe sound speed that is not positive counts as zero
    const double ct2 = fmax(gm1 * fma(-0.5, q2, Ht), 1e-280);
    const double ct = ct2 * rsq3(ct2);
    SL = fmin(uL - cL, ut - ct);
    SR = fmax(uR + cR, ut + ct);
  }
  const double gL = UL[0] * (SL - uL), gR = UR[0] * (SR - uR);
  const double num = fma(0.0, cL + cR, fma(gL, uL, fma(-gR, uR, pR - pL)));
  const double Ss = num * rcp3(gL - gR);
  const bool left = Ss >= 0.0;
  const double S = left ? SL : SR, rd = left ? gL : gR, u = left ? uL : uR, p = left ? pL : pR;
  const double e = left ? eL : eR, mK = left ? UL[1 + A] : UR[1 + A];
  const double iv = rcp3(S - Ss);
  const bool star = left ? S < 0.0 : S > 0.0;  // 0 between S_K and S*
  const double ik = star ? iv : 0.0, B = S * ik;
  const double f = fma(rd * ik, Ss, star ? 0.0 : mK);
  const double Aq = B * rd, q = Ss - u;
  F[0] = f;
#pragma unroll
  for (int b = 0; b < D; ++b)
    F[1 + b] = b == A ? fma(u, f, fma(Aq, q, p)) : f * (left ? vL[b] : vR[b]);
  F[D + 1] = fma(e, f, fma(p, u, q * fma(Aq, Ss, B * p)));
}

// Reverse sweep of hllc_line: for the cotangent G of the flux, GL = (dF/dUL)^T
// G and GR = (dF/dUR)^T G.  The forward values are formed with hllc_line's
// expressions, so the same side K, bounds and star branch are taken.  The
// sweep goes back to (rho, v, p, e = E / rho) of both sides and from there to
// the conserved variables; no branches (a divergent one would split the
// caller's code), a cotangent that belongs to one side only is selected for
// L and the rest is R's.
template <int D, int A, int FX>
__device__ __forceinline__ void hllc_line_vjp(const double (&UL)[D + 2], const double (&UR)[D + 2], double g,
                                              const double (&G)[D + 2], double (&GL)[D + 2], double (&GR)[D + 2]) {
  const double gm1 = g - 1.0;
  const double rsL = rsq3(UL[0]), rsR = rsq3(UR[0]);
  const double irL = rsL * rsL, irR = rsR * rsR;
  double vL[D], vR[D], keL = 0.0, keR = 0.0;  // |m|^2 / rho
#pragma unroll
  for (int b = 0; b < D; ++b) {
    vL[b] = UL[1 + b] * irL;
    vR[b] = UR[1 + b] * irR;
    keL = fma(UL[1 + b], vL[b], keL);
    keR = fma(UR[1 + b], vR[b], keR);
  }
  const double uL = vL[A], uR = vR[A];
  const double pL = gm1 * fma(-0.5, keL, UL[D + 1]), pR = gm1 * fma(-0.5, keR, UR[D + 1]);
  const double xL = g * pL * irL, xR = g * pR * irR;
  const double yL = rsq3(xL), yR = rsq3(xR);
  const double cL = xL * yL, cR = xR * yR;
  const double eL = UL[D + 1] * irL, eR = UR[D + 1] * irR;
  double SL, SR, is = 0.0, wL = 0.0, wR = 0.0, ct = 0.0, yt = 0.0, HL = 0.0, HR = 0.0, vt[D];
  bool lo2, hi2;  // the bound is the second operand of its min / max
  if constexpr (FX == DG_HLLC_DAVIS) {
    const double a = uL - cL, b = uR - cR, c = uL + cL, d = uR + cR;
    SL = fmin(a, b);
    SR = fmax(c, d);
    lo2 = b < a;
    hi2 = d > c;
  } else {
    const double sL = UL[0] * rsL, sR = UR[0] * rsR;
    is = rcp3(sL + sR);
    wL = sL * is;
    wR = sR * is;
    double q2 = 0.0;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      vt[b] = fma(wL, vL[b], wR * vR[b]);
      q2 = fma(vt[b], vt[b], q2);
    }
    HL = fma(pL, irL, eL);
    HR = fma(pR, irR, eR);
    const double ct2 = gm1 * fma(-0.5, q2, fma(wL, HL, wR * HR)), c2 = fmax(ct2, 1e-280);
    const double y = rsq3(c2);
    ct = c2 * y;
    yt = ct2 > 0.0 ? y : 0.0;
    const double a = uL - cL, b = vt[A] - ct, c = uR + cR, d = vt[A] + ct;
    SL = fmin(a, b);
    SR = fmax(c, d);
    lo2 = b < a;
    hi2 = d > c;
  }
  const double dL = SL - uL, dR = SR - uR, aL = UL[0] * dL, aR = UR[0] * dR;
  const double num = fma(0.0, cL + cR, fma(aL, uL, fma(-aR, uR, pR - pL)));
  const double iden = rcp3(aL - aR), Ss = num * iden;
  const bool left = Ss >= 0.0;
  const double S = left ? SL : SR, rho = left ? UL[0] : UR[0], u = left ? uL : uR, p = left ? pL : pR;
  const double e = left ? eL : eR, d = S - u, iv = rcp3(S - Ss), q = Ss - u;
  const bool star = left ? S < 0.0 : S > 0.0;
  const double ik = star ? iv : 0.0, B = S * ik, rd = left ? aL : aR, Aq = B * rd, si = Ss * iv;
  const double f = fma(rd * ik, Ss, star ? 0.0 : left ? UL[1 + A] : UR[1 + A]);

  // F_0 = f, F_n = u f + p + Aq q, F_t = v_t f, F_E = e f + p u + q (Aq S* + B p)
  double gf = fma(u, G[1 + A], fma(e, G[D + 1], G[0]));
  double gv[D];  // of side K's velocities
#pragma unroll
  for (int b = 0; b < D; ++b)
    if (b != A) {
      gf = fma(left ? vL[b] : vR[b], G[1 + b], gf);
      gv[b] = f * G[1 + b];
    }
  const double gE = G[D + 1], gn = G[1 + A], qE = q * gE;
  const double ge = f * gE;
  double gp = fma(B, qE, fma(u, gE, gn));
  const double gA = fma(Ss, qE, q * gn);
  const double gq = fma(Aq, gn, fma(Aq, Ss, B * p) * gE);
  double gSs = fma(Aq, qE, gq);
  double gu = fma(f, gn, fma(p, gE, -gq));
  const double gB = fma(p, qE, rd * gA);
  const double h = star ? gf : 0.0, hm = gf - h;  // the star form of f, and the momentum as f
  double grho = fma(B * d, gA, d * si * h);
  const double gd = fma(B * rho, gA, rho * si * h);
  gSs = fma(rd * iv, h, gSs);
  const double giv = fma(rd * Ss, h, star ? S * gB : 0.0);
  const double tS = -iv * iv * giv;
  double gS = (star ? iv * gB : 0.0) + gd + tS;
  gu -= gd;
  gSs -= tS;
  const double gnum = gSs * iden, gden = -gnum * Ss;
  // side K's share to L or R
  double rL = left ? grho : 0.0, rR = grho - rL, pgL = left ? gp : 0.0, pgR = gp - pgL;
  double sgL = left ? gS : 0.0, sgR = gS - sgL, egL = left ? ge : 0.0, egR = ge - egL;
  double gvL[D], gvR[D];
  gv[A] = gu;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    gvL[b] = left ? gv[b] : 0.0;
    gvR[b] = gv[b] - gvL[b];
  }
  // S* = num / den, num = p_R - p_L + a_L u_L - a_R u_R, den = a_L - a_R, a = rho (S - u)
  pgR += gnum;
  pgL -= gnum;
  const double gaL = fma(gnum, uL, gden), gaR = -fma(gnum, uR, gden);
  rL = fma(dL, gaL, rL);
  rR = fma(dR, gaR, rR);
  const double tL = UL[0] * gaL, tR = UR[0] * gaR;
  sgL += tL;
  sgR += tR;
  gvL[A] += fma(gnum, aL, -tL);
  gvR[A] -= fma(gnum, aR, tR);
  // wave-speed bounds
  double gcL, gcR;
  if constexpr (FX == DG_HLLC_DAVIS) {
    const double l1 = lo2 ? 0.0 : sgL, l2 = sgL - l1, h1 = hi2 ? 0.0 : sgR, h2 = sgR - h1;
    gvL[A] += l1 + h1;
    gvR[A] += l2 + h2;
    gcL = h1 - l1;
    gcR = h2 - l2;
  } else {
    const double l2 = lo2 ? sgL : 0.0, l1 = sgL - l2, h2 = hi2 ? sgR : 0.0, h1 = sgR - h2;
    gvL[A] += l1;
    gvR[A] += h1;
    gcL = -l1;
    gcR = h1;
    const double gHt = 0.5 * gm1 * (h2 - l2) * yt, gut = l2 + h2;
    double gw = (HL - HR) * gHt;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const double gb = fma(-vt[b], gHt, b == A ? gut : 0.0);
      gw = fma(vL[b] - vR[b], gb, gw);
      gvL[b] = fma(wL, gb, gvL[b]);
      gvR[b] = fma(wR, gb, gvR[b]);
    }
    // w_L = s_L / (s_L + s_R), s = sqrt(rho)
    const double gs = 0.5 * gw * is;
    rL = fma(gs * wR, rsL, rL);
    rR = fma(-gs * wL, rsR, rR);
    // H = e + p / rho
    const double hL = wL * gHt, hR = wR * gHt;
    egL += hL;
    egR += hR;
    pgL = fma(hL, irL, pgL);
    pgR = fma(hR, irR, pgR);
    rL = fma(-hL * pL, irL * irL, rL);
    rR = fma(-hR * pR, irR * irR, rR);
  }
  // c = sqrt(g p / rho)
  pgL = fma(0.5 * g * irL * yL, gcL, pgL);
  pgR = fma(0.5 * g * irR * yR, gcR, pgR);
  rL = fma(-0.5 * cL * irL, gcL, rL);
  rR = fma(-0.5 * cR * irR, gcR, rR);
  // to the conserved variables: p = gm1 (E - rho |v|^2 / 2), v = m / rho, e = E / rho
  const double kL = gm1 * pgL, kR = gm1 * pgR;
  GL[D + 1] = fma(irL, egL, kL);
  GR[D + 1] = fma(irR, egR, kR);
  double sL = -eL * egL, sR = -eR * egR;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    sL = fma(-vL[b], gvL[b], sL);
    sR = fma(-vR[b], gvR[b], sR);
    GL[1 + b] = fma(irL, gvL[b], -kL * vL[b]);
    GR[1 + b] = fma(irR, gvR[b], -kR * vR[b]);
  }
  GL[1 + A] += left ? hm : 0.0;
  GR[1 + A] += left ? 0.0 : hm;
  GL[0] = fma(irL, sL, fma(0.5 * keL * irL, kL, rL));
  GR[0] = fma(irR, sR, fma(0.5 * keR * irR, kR, rR));
}

// x of the lane below (lane 0 keeps its own) and of the lane above (lane 63
// keeps its own): whole-wave DPP shifts, no LDS
__device__ __forceinline__ double lane_below(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_above(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x130, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x130, 0xf, 0xf, false));
}

}  // namespace dg
