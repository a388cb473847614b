// Device code shared by the kernels' source files: shapes, grids, reciprocals,
// the time-step rate, the Euler flux, the Riemann solver and its derivative,
// the stage combination and the mode order.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dg_internal.h"

namespace dg {

template <int D, int K>
struct Cfg {
  static constexpr int NV = D + 2;
  static constexpr int N1 = K + 1;
  static constexpr int N = D == 2 ? (K + 1) * (K + 2) / 2 : (K + 1) * (K + 2) * (K + 3) / 6;
  static constexpr int Q = D == 2 ? N1 * N1 : N1 * N1 * N1;
  static constexpr int QF = Q / N1;
  static constexpr int M = (K + 4) / 2 < 2 ? 2 : (K + 4) / 2;
  static constexpr int NS = D * M * QF;
  static constexpr int B = 0;
  static constexpr int DW = B + Q * N;
  static constexpr int TF = DW + D * Q * N;
  static constexpr int TW = TF + D * 2 * QF * N;
  static constexpr int WQ = TW + D * 2 * QF * N;
  static constexpr int PS = WQ + Q;
  static constexpr int XQ = PS + NS * N;
  static constexpr int HG = XQ + 3 * Q;
  static constexpr int HW = HG + D * 2 * 4 * QF * N;
  static constexpr int TOTAL = HW + D * 2 * 4 * QF * N;
};

struct Grid {
  int nx, ny, nz;
  long ncell;
  int bc[3];
  double fac;    // (2/dx) 2^-d
  double gamma;
  // block order of the 3D MFMA stage kernel (block_order): strips of xg
  // blocks, xzc planes per XCD, xp blocks per plane; xg = 0: launch order
  int xg, xzc, xp;
};

// The launch's blocks go to the eight XCDs in turn (block b to XCD b mod 8),
// each XCD with its own L2.  For a 3D grid of whole 64-cell blocks per plane
// (xp of them) and a multiple of eight planes, XCD x takes the planes
// [x xzc, (x + 1) xzc), and its j-th block is strip lo of plane zz of
// strip row hi, strips (xg blocks, one x-row when the row is whole blocks)
// fastest, then the planes, then the strip rows: a block's z neighbours ran
// xg blocks earlier on the same XCD and its y neighbours xg xzc blocks
// earlier, so both are mostly still in that XCD's L2 (in launch order the
// y neighbours sit on another XCD).  A permutation of the blocks whatever
// the dispatch does.
__device__ inline long block_order(const Grid &g, long b) {
  if (g.xg == 0) return b;
  const long x = b & 7, j = b >> 3;
  const long lo = j % g.xg, r = j / g.xg;
  const long zz = r % g.xzc, hi = r / g.xzc;
  return (x * g.xzc + zz) * g.xp + hi * g.xg + lo;
}

enum : int { FLAG_NEGATIVE = 1, FLAG_NAN = 2 };

// Flat index of the neighbour of (ix,iy,iz) along axis a in direction dir,
// or -1 at a transmissive boundary.
__device__ inline long neighbour(const Grid &g, int ix, int iy, int iz, int a, int dir) {
  int i[3] = {ix, iy, iz};
  int n[3] = {g.nx, g.ny, g.nz};
  i[a] += dir;
  if (i[a] < 0 || i[a] >= n[a]) {
    if (g.bc[a] == DG_BC_TRANSMISSIVE) return -1;
    i[a] = i[a] < 0 ? i[a] + n[a] : i[a] - n[a];
  }
  return ((long)i[2] * g.ny + i[1]) * g.nx + i[0];
}

// Reciprocal and reciprocal square root from the hardware estimates plus
// Newton steps (within an ulp or two; the IEEE-rounded division and square
// root expand into much longer dependent sequences).  Used by the Riemann
// solver and the volume flux.
__device__ inline double vrcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ inline double vrsq(double x) {
  double y = __builtin_amdgcn_rsq(x);
  // y <- y (3 - x y^2) / 2, twice
  double h = 0.5 * x;
  double t = fma(-h, y * y, 0.5);
  y = fma(y, t, y);
  t = fma(-h, y * y, 0.5);
  return fma(y, t, y);
}
__device__ inline float vrcp(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}
__device__ inline float vrsq(float x) {
  float y = __builtin_amdgcn_rsqf(x);
  return fmaf(y, fmaf(-0.5f * x, y * y, 0.5f), y);
}

// Signal rate sum_a (|v_a| + c)/dx of a cell mean U (eq. time_step); `bad`
// records a non-positive density or pressure.  Shared by every kernel that
// forms the time step, so that all of them obtain bitwise the same rate.
template <int D>
__device__ inline double cell_rate(const double *U, double gamma, double dx, bool &bad, double gk = 0.0,
                                   double amax = 0.0) {
  double ke = 0.0;
#pragma unroll
  for (int b = 0; b < D; ++b) ke += U[1 + b] * U[1 + b] / U[0];
  const double p = (gamma - 1.0) * (U[D + 1] - 0.5 * ke);
  bad |= !(U[0] > 0.0) || !(p > 0.0);
  const double c = sqrt(gamma * p / U[0]);
  double rate = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) rate += (fabs(U[1 + a] / U[0]) + c) / dx;
  // gravity step (Sec. 2.5) dt <= c / (sqrt(2 gamma (gamma-1)) |grad Phi|) as a
  // rate against the same CFL f_k: gk = CFL f_k sqrt(2 gamma (gamma-1))
  if (amax > 0.0) rate = fmax(rate, gk * amax / c);
  return rate;
}

// maximum over the 64 lanes of a wave (all lanes active)
__device__ inline double wave_max(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off));
  return x;
}

// The maximum signal rate is reduced into RATE_SLOTS 64-bit words, one per
// 128-byte line, each holding the bit pattern of a non-negative double (such
// doubles order like their bits, so atomicMax on the pattern is a max); the
// rate is the largest slot.  Workgroup b folds into slot b mod 8, i.e. one
// slot per XCD: a single word taking every workgroup's atomic serialises
// them.
constexpr int RATE_SLOTS = 8, RATE_STRIDE = 16;
static_assert(RATE_SLOTS * RATE_STRIDE == DG_RATE_STATE, "layout of the carried rate state");
__device__ inline unsigned long long *rate_slot(unsigned long long *w, int b) {
  return w + RATE_STRIDE * (b % RATE_SLOTS);
}

// Time-step work that the fused SSP-RK3 step hands to the stage kernels
// (see k_rhs_tile2d); `word` is the carried rate state (RATE_SLOTS slots).
enum : int { RATE_NONE = 0, RATE_DT = 1, RATE_CLEAR = 2, RATE_FOLD = 3 };
struct RateOp {
  unsigned long long *word;
  double *dt_out;
  double cfl_fk;  // CFL times the order factor of the time step
  double dx;
  int op;
  const double *gmax = nullptr;  // per cell the largest |grad Phi| at its nodes (gravity), or null
  double gk = 0.0;               // CFL f_k sqrt(2 gamma (gamma-1))
};

// Euler flux f_a(U) (eq. flux_vectors; 2D drops the third velocity).
template <int D, class R>
__device__ inline void euler_flux(const R *U, int a, R gm1, R *F) {
  const R ir = vrcp(U[0]);
  R ke = R(0);
#pragma unroll
  for (int b = 0; b < D; ++b) ke = fma(U[1 + b], U[1 + b] * ir, ke);
  const R p = gm1 * (U[D + 1] - R(0.5) * ke);
  const R va = U[1 + a] * ir;
  F[0] = U[1 + a];
#pragma unroll
  for (int b = 0; b < D; ++b) F[1 + b] = fma(U[1 + b], va, b == a ? p : R(0));
  F[D + 1] = (U[D + 1] + p) * va;
}

// Scalar helpers so that the Riemann solver runs on doubles and on floats
// with the same sequence of operations.
__device__ inline double vfma(double a, double b, double c) { return fma(a, b, c); }
__device__ inline double vsqrt(double a) { return sqrt(a); }
__device__ inline double vmin(double a, double b) { return b < a ? b : a; }
__device__ inline double vmax(double a, double b) { return b > a ? b : a; }
__device__ inline double val(double a) { return a; }
__device__ inline float vfma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ inline float vsqrt(float a) { return sqrtf(a); }
__device__ inline float vmin(float a, float b) { return b < a ? b : a; }
__device__ inline float vmax(float a, float b) { return b > a ? b : a; }
__device__ inline double val(float a) { return a; }


template <class T>
__device__ inline T cst(double x);
template <>
__device__ inline double cst<double>(double x) { return x; }
template <>
__device__ inline float cst<float>(double x) { return (float)x; }

// HLLC numerical flux in +a between traces UL (low side) and UR (high side),
// in the compact form F = F_K + S_K^(-/+) (U*_K - U_K) with K = L if S* >= 0
// (S_L^- = min(S_L, 0)) and K = R otherwise (S_R^+ = max(S_R, 0)); this
// equals the four-region selection of the textbook solver.  Wave-speed
// bounds: Einfeldt-Batten (Roe-averaged, FX = 0) or Davis (FX = 1).
//
// The choice is a template parameter, not a run-time flag: with a uniform
// flag branched on inside loops that run under different exec masks (the
// hanging sub-faces of the refined box), the compiler built the flag's lane
// mask under one exec mask and reused it under another, so lanes that had
// been inactive took the other branch.
template <class T, int D, int FX, bool SEL = false>
__device__ inline void hllc(const T *UL, const T *UR, int a, double g, T *F) {
  // The normal axis a may be a run-time value: components are picked with
  // unrolled compares (no dynamic register indexing).  One reciprocal square
  // root per side gives sqrt(rho) and 1/rho.  SEL: every arm of a
  // conditional is evaluated and the result selected, so the solver contains
  // no branch (a conditional with a costly arm otherwise becomes a divergent
  // branch, which splits the caller's code into separately scheduled blocks;
  // the one-thread-per-cell kernels run faster with the branches).  The
  // results are the same bit for bit.
  const T gm1 = cst<T>(g - 1.0), gg = cst<T>(g), half = cst<T>(0.5);
  const T zero = cst<T>(0.0);
  const T rsL = vrsq(UL[0]), rsR = vrsq(UR[0]);
  const T irL = rsL * rsL, irR = rsR * rsR;
  T vL[D], vR[D], keL = zero, keR = zero, uL = zero, uR = zero, mL = zero, mR = zero;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    vL[b] = UL[1 + b] * irL;
    vR[b] = UR[1 + b] * irR;
    keL = vfma(UL[1 + b], vL[b], keL);
    keR = vfma(UR[1 + b], vR[b], keR);
    if (b == a) {
      uL = vL[b];
      uR = vR[b];
      mL = UL[1 + b];
      mR = UR[1 + b];
    }
  }
  const T pL = gm1 * (UL[D + 1] - half * keL);
  const T pR = gm1 * (UR[D + 1] - half * keR);
  // c = sqrt(g p / rho) = g p rsq(g p rho)
  const T gpL = gg * pL, gpR = gg * pR;
  const T cL = gpL * vrsq(gpL * UL[0]), cR = gpR * vrsq(gpR * UR[0]);
  T SL, SR;
  if constexpr (FX == DG_HLLC_DAVIS) {
    SL = vmin(uL - cL, uR - cR);
    SR = vmax(uL + cL, uR + cR);
  } else {
    const T sL = UL[0] * rsL, sR = UR[0] * rsR;
    const T is = vrcp(sL + sR);
    T q2 = zero, ut = zero;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const T vt = (sL * vL[b] + sR * vR[b]) * is;
      q2 = vfma(vt, vt, q2);
      if (b == a) ut = vt;
    }
    const T HL = (UL[D + 1] + pL) * irL, HR = (UR[D + 1] + pR) * irR;
    const T Ht = (sL * HL + sR * HR) * is;
    const T ct2 = gm1 * (Ht - half * q2);
    T ct;
    if constexpr (SEL) {
      const T rq = vrsq(ct2);
      ct = val(ct2) > 0.0 ? ct2 * rq : zero;
    } else {
      ct = val(ct2) > 0.0 ? ct2 * vrsq(ct2) : zero;
    }
    SL = vmin(uL - cL, ut - ct);
    SR = vmax(uR + cR, ut + ct);
  }
  const T dL = SL - uL, dR = SR - uR;
  const T Ss = (pR - pL + mL * dL - mR * dR) * vrcp(UL[0] * dL - UR[0] * dR);
  const bool left = val(Ss) >= 0.0;
  T U[D + 2];
#pragma unroll
  for (int v = 0; v < D + 2; ++v) U[v] = left ? UL[v] : UR[v];
  const T SK = left ? SL : SR;
  T SKc;
  if constexpr (SEL) {
    const T SLc = vmin(SL, zero), SRc = vmax(SR, zero);
    SKc = left ? SLc : SRc;
  } else {
    SKc = left ? vmin(SL, zero) : vmax(SR, zero);
  }
  const T irK = left ? irL : irR, pK = left ? pL : pR;
  const T uK = left ? uL : uR, dK = left ? dL : dR, mK = left ? mL : mR;
  T FK[D + 2];
  // physical flux of the selected side
  FK[0] = mK;
#pragma unroll
  for (int b = 0; b < D; ++b) FK[1 + b] = vfma(U[1 + b], uK, b == a ? pK : zero);
  FK[D + 1] = (U[D + 1] + pK) * uK;
  // star state rho_K (S_K - u_K)/(S_K - S*) (1, S* n + v_t, E_K/rho_K + (S* - u_K)(S* + p_K/(rho_K (S_K - u_K))))
  // with r = rho_K (S_K - u_K) and f = r / (S_K - S*): f p_K / r = p_K / (S_K - S*)
  const T ivS = vrcp(SK - Ss);
  const T fac = (U[0] * dK) * ivS;
  T Us[D + 2];
  Us[0] = fac;
#pragma unroll
  for (int b = 0; b < D; ++b) Us[1 + b] = fac * (b == a ? Ss : U[1 + b] * irK);
  Us[D + 1] = vfma(fac, vfma(Ss - uK, Ss, U[D + 1] * irK), (Ss - uK) * pK * ivS);
#pragma unroll
  for (int v = 0; v < D + 2; ++v) F[v] = vfma(SKc, Us[v] - U[v], FK[v]);
}

// Reverse-mode derivative of hllc<double, D, FX>: for the cotangent gF of the
// flux, gUL = (dF/dUL)^T gF and gUR = (dF/dUR)^T gF.  The forward values are
// recomputed with the same expressions as hllc, so every branch (the
// wave-speed bounds, S* >= 0, the min/max against 0) is taken as there; one
// forward and one reverse sweep give both sides' rows at once.
template <int D, int FX>
__device__ inline void hllc_vjp(const double *UL, const double *UR, int a, double g, const double *gF,
                                double *gUL, double *gUR) {
  constexpr int NV = D + 2;
  const double gm1 = g - 1.0;
  // ---- forward
  const double rsL = vrsq(UL[0]), rsR = vrsq(UR[0]);
  const double irL = rsL * rsL, irR = rsR * rsR;
  double vL[D], vR[D], keL = 0.0, keR = 0.0, uL = 0.0, uR = 0.0, mL = 0.0, mR = 0.0;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    vL[b] = UL[1 + b] * irL;
    vR[b] = UR[1 + b] * irR;
    keL = fma(UL[1 + b], vL[b], keL);
    keR = fma(UR[1 + b], vR[b], keR);
    if (b == a) {
      uL = vL[b];
      uR = vR[b];
      mL = UL[1 + b];
      mR = UR[1 + b];
    }
  }
  const double pL = gm1 * (UL[D + 1] - 0.5 * keL);
  const double pR = gm1 * (UR[D + 1] - 0.5 * keR);
  const double kpL = g * pL, kpR = g * pR;  // gamma p
  const double yL = vrsq(kpL * UL[0]), yR = vrsq(kpR * UR[0]);
  const double cL = kpL * yL, cR = kpR * yR;
  double SL, SR;
  bool sl2, sr2;  // the min/max took its second operand
  double sL = 0.0, sR = 0.0, is = 0.0, vt[D], q2 = 0.0, ut = 0.0, HL = 0.0, HR = 0.0, ct2 = 0.0, ct = 0.0;
#pragma unroll
  for (int b = 0; b < D; ++b) vt[b] = 0.0;
  if constexpr (FX == DG_HLLC_DAVIS) {
    const double x1 = uL - cL, y1 = uR - cR, x2 = uL + cL, y2 = uR + cR;
    sl2 = y1 < x1;
    sr2 = y2 > x2;
    SL = sl2 ? y1 : x1;
    SR = sr2 ? y2 : x2;
  } else {
    sL = UL[0] * rsL;
    sR = UR[0] * rsR;
    is = vrcp(sL + sR);
#pragma unroll
    for (int b = 0; b < D; ++b) {
      vt[b] = (sL * vL[b] + sR * vR[b]) * is;
      q2 = fma(vt[b], vt[b], q2);
      if (b == a) ut = vt[b];
    }
    HL = (UL[D + 1] + pL) * irL;
    HR = (UR[D + 1] + pR) * irR;
    const double Ht = (sL * HL + sR * HR) * is;
    ct2 = gm1 * (Ht - 0.5 * q2);
    ct = ct2 > 0.0 ? ct2 * vrsq(ct2) : 0.0;
    const double x1 = uL - cL, y1 = ut - ct, x2 = uR + cR, y2 = ut + ct;
    sl2 = y1 < x1;
    sr2 = y2 > x2;
    SL = sl2 ? y1 : x1;
    SR = sr2 ? y2 : x2;
  }
  const double dL = SL - uL, dR = SR - uR;
  const double iden = vrcp(UL[0] * dL - UR[0] * dR);
  const double Ss = (pR - pL + mL * dL - mR * dR) * iden;
  const bool left = Ss >= 0.0;
  double UK[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) UK[v] = left ? UL[v] : UR[v];
  const double SK = left ? SL : SR;
  const bool pass = left ? !(0.0 < SL) : !(0.0 > SR);  // S_K^-/+ equals S_K (else 0)
  const double SKc = pass ? SK : 0.0;
  const double irK = left ? irL : irR, pK = left ? pL : pR, uK = left ? uL : uR, dK = left ? dL : dR;
  const double ivS = vrcp(SK - Ss);
  const double fac = (UK[0] * dK) * ivS;
  const double A = fma(Ss - uK, Ss, UK[D + 1] * irK);
  double Us[NV];
  Us[0] = fac;
#pragma unroll
  for (int b = 0; b < D; ++b) Us[1 + b] = fac * (b == a ? Ss : UK[1 + b] * irK);
  Us[D + 1] = fma(fac, A, (Ss - uK) * pK * ivS);

  // ---- reverse: F = F_K + SKc (Us - U_K)
  double gUK[NV], gSKc = 0.0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    gSKc = fma(gF[v], Us[v] - UK[v], gSKc);
    gUK[v] = -SKc * gF[v];
  }
  double gfac = SKc * gF[0], gSs = 0.0, guK = 0.0, girK = 0.0, gpK = 0.0, givS = 0.0;
#pragma unroll
  for (int b = 0; b < D; ++b) {
    const double gu = SKc * gF[1 + b];
    if (b == a) {
      gfac = fma(gu, Ss, gfac);
      gSs = fma(gu, fac, gSs);
    } else {
      gfac = fma(gu, UK[1 + b] * irK, gfac);
      gUK[1 + b] = fma(gu, fac * irK, gUK[1 + b]);
      girK = fma(gu, fac * UK[1 + b], girK);
    }
  }
  {
    const double ge = SKc * gF[D + 1];
    gfac = fma(ge, A, gfac);
    const double gA = ge * fac;
    gSs = fma(gA, 2.0 * Ss - uK, gSs);
    guK = fma(-gA, Ss, guK);
    gUK[D + 1] = fma(gA, irK, gUK[D + 1]);
    girK = fma(gA, UK[D + 1], girK);
    const double t = Ss - uK, gt = ge * pK * ivS;
    gpK = fma(ge, t * ivS, gpK);
    givS = fma(ge, t * pK, givS);
    gSs += gt;
    guK -= gt;
  }
  // fac = rho_K d_K ivS, ivS = 1/(S_K - S*)
  gUK[0] = fma(gfac, dK * ivS, gUK[0]);
  double gdK = gfac * UK[0] * ivS;
  givS = fma(gfac, UK[0] * dK, givS);
  double gSK = -givS * ivS * ivS;
  gSs = fma(givS, ivS * ivS, gSs);
  // F_K
  gUK[1 + a] += gF[0];
#pragma unroll
  for (int b = 0; b < D; ++b) {
    gUK[1 + b] = fma(gF[1 + b], uK, gUK[1 + b]);
    guK = fma(gF[1 + b], UK[1 + b], guK);
  }
  gpK += gF[1 + a];
  gUK[D + 1] = fma(gF[D + 1], uK, gUK[D + 1]);
  gpK = fma(gF[D + 1], uK, gpK);
  guK = fma(gF[D + 1], UK[D + 1] + pK, guK);
  if (pass) gSK += gSKc;
  // d_K = S_K - u_K
  gSK += gdK;
  guK -= gdK;
  // the K side back to L or R
  double gSL = left ? gSK : 0.0, gSR = left ? 0.0 : gSK;
  double gpL = left ? gpK : 0.0, gpR = left ? 0.0 : gpK;
  double guL = left ? guK : 0.0, guR = left ? 0.0 : guK;
  double girL = left ? girK : 0.0, girR = left ? 0.0 : girK;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    gUL[v] = left ? gUK[v] : 0.0;
    gUR[v] = left ? 0.0 : gUK[v];
  }
  // S* = num / den
  const double gnum = gSs * iden, gden = -gSs * Ss * iden;
  gpR += gnum;
  gpL -= gnum;
  gUL[1 + a] = fma(gnum, dL, gUL[1 + a]);
  gUR[1 + a] = fma(-gnum, dR, gUR[1 + a]);
  double gdL = fma(gnum, mL, gden * UL[0]);
  double gdR = fma(-gnum, mR, -gden * UR[0]);
  gUL[0] = fma(gden, dL, gUL[0]);
  gUR[0] = fma(-gden, dR, gUR[0]);
  gSL += gdL;
  guL -= gdL;
  gSR += gdR;
  guR -= gdR;
  // wave-speed bounds
  double gcL = 0.0, gcR = 0.0;
  if constexpr (FX == DG_HLLC_DAVIS) {
    if (sl2) { guR += gSL; gcR -= gSL; } else { guL += gSL; gcL -= gSL; }
    if (sr2) { guR += gSR; gcR += gSR; } else { guL += gSR; gcL += gSR; }
  } else {
    double gut = 0.0, gct = 0.0;
    if (sl2) { gut += gSL; gct -= gSL; } else { guL += gSL; gcL -= gSL; }
    if (sr2) { gut += gSR; gct += gSR; } else { guR += gSR; gcR += gSR; }
    const double gct2 = ct2 > 0.0 ? 0.5 * gct * vrsq(ct2) : 0.0;
    const double gHt = gct2 * gm1, gq2 = -0.5 * gm1 * gct2;
    double gsL = gHt * HL * is, gsR = gHt * HR * is, gis = gHt * (sL * HL + sR * HR);
    const double gHL = gHt * sL * is, gHR = gHt * sR * is;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const double gv = fma(2.0 * vt[b], gq2, b == a ? gut : 0.0);
      gsL = fma(gv, vL[b] * is, gsL);
      gsR = fma(gv, vR[b] * is, gsR);
      gis = fma(gv, sL * vL[b] + sR * vR[b], gis);
      // vt depends on vL, vR: folded into the velocity gradients below
      gUL[1 + b] = fma(gv * sL * is, irL, gUL[1 + b]);
      girL = fma(gv * sL * is, UL[1 + b], girL);
      gUR[1 + b] = fma(gv * sR * is, irR, gUR[1 + b]);
      girR = fma(gv * sR * is, UR[1 + b], girR);
    }
    gsL = fma(-gis, is * is, gsL);
    gsR = fma(-gis, is * is, gsR);
    // H = (E + p) / rho
    gUL[D + 1] = fma(gHL, irL, gUL[D + 1]);
    gpL = fma(gHL, irL, gpL);
    girL = fma(gHL, UL[D + 1] + pL, girL);
    gUR[D + 1] = fma(gHR, irR, gUR[D + 1]);
    gpR = fma(gHR, irR, gpR);
    girR = fma(gHR, UR[D + 1] + pR, girR);
    // s = sqrt(rho)
    gUL[0] = fma(gsL, 0.5 * rsL, gUL[0]);
    gUR[0] = fma(gsR, 0.5 * rsR, gUR[0]);
  }
  // c = sqrt(g p / rho): dc/dp = g y / 2, dc/drho = -c / (2 rho)
  gpL = fma(gcL, 0.5 * g * yL, gpL);
  gUL[0] = fma(-gcL, 0.5 * cL * irL, gUL[0]);
  gpR = fma(gcR, 0.5 * g * yR, gpR);
  gUR[0] = fma(-gcR, 0.5 * cR * irR, gUR[0]);
  // u = m_a / rho (as v_a); p = gm1 (E - ke/2), ke = sum m_b v_b, v_b = m_b / rho
  const double gkeL = -0.5 * gm1 * gpL, gkeR = -0.5 * gm1 * gpR;
  gUL[D + 1] = fma(gm1, gpL, gUL[D + 1]);
  gUR[D + 1] = fma(gm1, gpR, gUR[D + 1]);
#pragma unroll
  for (int b = 0; b < D; ++b) {
    const double gvL = fma(gkeL, UL[1 + b], b == a ? guL : 0.0);
    const double gvR = fma(gkeR, UR[1 + b], b == a ? guR : 0.0);
    gUL[1 + b] = fma(gkeL, vL[b], fma(gvL, irL, gUL[1 + b]));
    gUR[1 + b] = fma(gkeR, vR[b], fma(gvR, irR, gUR[1 + b]));
    girL = fma(gvL, UL[1 + b], girL);
    girR = fma(gvR, UR[1 + b], girR);
  }
  // ir = 1 / rho
  gUL[0] = fma(-girL, irL * irL, gUL[0]);
  gUR[0] = fma(-girR, irR * irR, gUR[0]);
}

// ---------------------------------------------------------------------------
// One stage of the time integrator in Shu-Osher form (App. D): with u the
// stage input, out = cu u + cl dt L(u) + sum_k a_k y_k over earlier stage
// values y_k (the stage values of an explicit Runge-Kutta tableau; SSP-RK3 is
// cu = cl = 1, then 1/4, 1/4 with 3/4 w^n, then 2/3, 2/3 with 1/3 w^n).
// ---------------------------------------------------------------------------
constexpr int MIX_MAX = 4;
struct Mix {
  const double *y[MIX_MAX];
  double a[MIX_MAX];
  double cu, cl;
  int n;
};

// the terms k >= k0 of the sum, added to o
__device__ inline double mix_tail(const Mix &m, double o, long i, int k0) {
#pragma unroll
  for (int k = 0; k < MIX_MAX; ++k)
    if (k >= k0 && k < m.n) o = fma(m.a[k], m.y[k][i], o);
  return o;
}

__device__ inline double mix_out(const Mix &m, double u, double L, double cldt, long i) {
  return mix_tail(m, fma(cldt, L, m.cu * u), i, 0);
}

// The refined box's geometry (see k_rhs_amr below).
struct AmrGrid {
  int n[3];    // base (coarse) grid
  int lo[3], hi[3];
  int nf[3];   // fine block
  long ncc, ncf;
  int bc[3];
  double facc, facf, dxc, dxf;
  double gamma;
};

template <int D>
__device__ inline bool amr_in_hole(const AmrGrid &g, const int *i) {
#pragma unroll
  for (int a = 0; a < D; ++a)
    if (i[a] < g.lo[a] || i[a] >= g.hi[a]) return false;
  return true;
}

// base-grid neighbour along a (periodic); false at a transmissive wall
template <int D>
__device__ inline bool amr_coarse_nb(const AmrGrid &g, const int *i, int a, int dir, int *j) {
#pragma unroll
  for (int b = 0; b < 3; ++b) j[b] = i[b];
  j[a] += dir;
  if (j[a] < 0 || j[a] >= g.n[a]) {
    if (g.bc[a] == DG_BC_TRANSMISSIVE) return false;
    j[a] = j[a] < 0 ? j[a] + g.n[a] : j[a] - g.n[a];
  }
  return true;
}

// Exponent of axis a in mode l (modes ordered by total degree, then
// x-exponent descending, then y-exponent descending).
template <int D>
__host__ __device__ constexpr int mode_exp(int l, int a) {
  int n = 0;
  for (int t = 0; t <= 8; ++t)
    for (int ex = t; ex >= 0; --ex)
      for (int ey = t - ex; ey >= 0; --ey) {
        const int ez = t - ex - ey;
        if (D == 2 && ez > 0) continue;
        if (n == l) return a == 0 ? ex : a == 1 ? ey : ez;
        ++n;
      }
  return 0;
}

static_assert(mode_exp<3>(1, 0) == 1 && mode_exp<3>(2, 1) == 1 && mode_exp<3>(3, 2) == 1 && mode_exp<3>(4, 0) == 2 &&
                  mode_exp<3>(5, 1) == 1 && mode_exp<3>(6, 2) == 1 && mode_exp<3>(9, 2) == 2 && mode_exp<2>(3, 0) == 2 &&
                  mode_exp<2>(5, 1) == 2 && mode_exp<3>(10, 0) == 3,
              "mode order: total degree, then x-exponent descending, then y-exponent descending");

// f(std::integral_constant<int, I>) for I = B .. E-1: the mode index is a
// compile-time constant, so register arrays indexed by a mode's exponents
// stay in registers
template <int B, int E, class F>
__device__ inline void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Quadtree mesh tables (built on the host by dg_tree_set).
struct TreeGrid {
  long nleaf;
  const int *lev;   // [nleaf]
  const int *info;  // [4][nleaf]: kind | sub << 2 | ch << 3, side 2a + s (ch: kind 3's child for the limiters)
  const int *nb;    // [8][nleaf]: neighbour (2 side + half)
  const int *grp;   // [4][nleaf]: the four leaves of this leaf's sibling group (child order), or -1
  double fac0;      // (2/dx) 2^-d of level 0
  double dx0;
  double gamma;
};

// Stage kernels of the other source files.  launch_line runs the stage on one
// of them and sets *err (a hipError_t) if its rule takes the context's grid,
// else it returns false.
bool launch_line(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                 const RateOp &ro, hipStream_t s, int *err);
bool split2d_takes(const dg_ctx *c);
int launch_split2d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                   const RateOp &ro, hipStream_t s);
int launch_split_tree(const dg_ctx *c, const TreeGrid &g, const double *w, double *out, const double *dt, int mode,
                      const Mix &mx, hipStream_t s);
int launch_adjoint2d(const dg_ctx *c, const double *w, const double *lam, const double *acc, double *out,
                     double *acc_out, const double *dt, int mode, double ca, double cb, hipStream_t s);
bool split3d_takes(const dg_ctx *c);
int launch_split3d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                   hipStream_t s);
bool march3d_takes(const dg_ctx *c);
int launch_march3d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                   hipStream_t s);

}  // namespace dg
