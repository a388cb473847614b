// Discrete adjoint of the 2D right-hand side and stages, a cell's work split
// over four waves (FP64).
#include "dg_march.h"

namespace dg {

struct AdjointGrid {
  int nx, ny;
  long nc;
  int wall[2];
  double fac, gamma;
  long columns;  // (nx + 1) ny
};

// G = sum_a J_a(U)^T Lam_a of the Euler fluxes f_x, f_y
__device__ __forceinline__ void flux_vjp2(const double (&U)[4], const double (&Lx)[4], const double (&Ly)[4], double g,
                                          double (&G)[4]) {
  const double gm1 = g - 1.0, ir = rcp3(U[0]);
  const double vx = U[1] * ir, vy = U[2] * ir, q2 = fma(vx, vx, vy * vy);
  const double hk = 0.5 * gm1 * q2, H = fma(gm1, fma(-0.5, fma(U[1], vx, U[2] * vy), U[3]), U[3]) * ir;
  const double lvx = fma(Lx[1], vx, Lx[2] * vy), lvy = fma(Ly[1], vx, Ly[2] * vy);
  const double sx = fma(Lx[3], vx, Lx[1]), sy = fma(Ly[3], vy, Ly[2]);  // la + lE va
  const double gs = gm1 * (sx + sy);
  G[0] = hk * (Lx[1] + Ly[2]) - vx * lvx - vy * lvy + (hk - H) * fma(Lx[3], vx, Ly[3] * vy);
  G[1] = fma(Lx[3], H, Lx[0] + lvx) + fma(Lx[1], vx, Ly[1] * vy) - gs * vx;
  G[2] = fma(Ly[3], H, Ly[0] + lvy) + fma(Ly[2], vy, Lx[2] * vx) - gs * vy;
  G[3] = fma(gm1, Lx[1] + Ly[2], g * fma(Lx[3], vx, Ly[3] * vy));
}

// mu_l += P~_n(+-1) m_t: the transpose of edge_coefs
template <int K, int A, int S>
__device__ __forceinline__ void edge_coefs_t(const double (&m)[K + 1], double (&mu)[(K + 1) * (K + 2) / 2]) {
  constexpr Line<K> L{};
  static_for<0, (K + 1) * (K + 2) / 2>([&](auto L_) {
    constexpr int l = decltype(L_)::value, ex = mode_exp<2>(l, 0), ey = mode_exp<2>(l, 1);
    constexpr int n = A == 0 ? ex : ey, t = A == 0 ? ey : ex;
    constexpr double s = (S == 0 && n % 2 ? -1.0 : 1.0) * L.b[n];
    mu[l] = fma(m[t], s, mu[l]);
  });
}

// The forward kernel's split (k_rhs_split2d) of the transposed operator: wave
// 0 the volume term, mu_l += sum_q phi_l(q) sum_a J_a^T Lam_a with Lam_a(q) = w_q
// d(lam)/d xi_a, waves 1, 2, 3 the x low, y low and y high faces: with g = w_r
// (lam_high - lam_low) on the face, one reverse sweep through the Riemann
// solver gives both cells' (dF/dU)^T g, of which an x face serves both (the
// lane below's through LDS) and a y face its own.  After one barrier wave v
// lifts variable v's four faces and applies the transposed stage.
// A face wave's registers are what limits it (a sweep holds about 60 values):
// one point at a time, the cotangent and the lane below's moments in LDS, two
// waves a SIMD.  Bound at k = 3 by the loads (a face wave reads 160 coefficients,
// 15 cycles of the load unit each) and the FP64 rate (four sweeps of 320
// operations) in about equal parts, behind them HBM (420 MB at 512^2, 80 us).
// A stage, four lanes per cell with every face swept from both sides before:
// k = 3, 32^2 29.0 -> 14.2, 256^2 80 -> 58, 512^2 320 -> 241 us; k = 2, 256^2
// 59 -> 31; k = 1, 64^2 12.1 -> 8.4, 512^2 135 -> 59.
template <int K, int FX, class Buf>
__global__ __launch_bounds__(256, 2) void k_adjoint_split2d(
    const double *__restrict__ w, const double *__restrict__ lam, const double *acc_in, double *__restrict__ out,
    double *acc_out, const double *__restrict__ dtp, AdjointGrid g, int mode, double ca, double cb,
    int *__restrict__ flag) {
  constexpr int N = (K + 1) * (K + 2) / 2, NM = K * (K + 1) / 2, n1 = K + 1;
  constexpr Line<K> L{};
  using Cell = typename Buf::Cell;
  using Off = typename Buf::Off;
  __shared__ double sv[4 * N * 64];           // [v][l][lane]: the cell's weights, then its volume term
  __shared__ double sd[4 * 2 * NM * 64];      // [v][axis][j][lane]: d(lam)/d xi_a
  __shared__ double sm[4 * 4 * n1 * 64];      // [x low (own), x low (below), y low, y high][v][e][lane]
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = gridDim.x, xcd = blockIdx.x % 8, jb = blockIdx.x / 8;
  const long blk = (long)xcd * (nb / 8) + min(xcd, nb % 8) + jb;
  const long e0 = 63 * blk + lane;
  const long e = min(e0, g.columns - 1);
  const int px = (int)(e % (g.nx + 1)), iy = (int)(e / (g.nx + 1));
  const bool own = px < g.nx && lane < 63 && e0 < g.columns;
  const Buf ws(w, g.nc, 4 * N), ls(lam, g.nc, 4 * N);
  const Cell nx8 = (Cell)8 * (Cell)g.nx, row = (Cell)iy * nx8;
  const Cell cell = row + (Cell)8 * (Cell)(px < g.nx ? px : 0);

  if (role == 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double x[1][N], y[1][N];
      load_cell<1, N>(ws, cell, x, (Off)(v * N) * ws.plane);
      load_cell<1, N>(ls, cell, y, (Off)(v * N) * ls.plane);
#pragma unroll
      for (int l = 0; l < N; ++l) sv[(v * N + l) * 64 + lane] = x[0][l];
      static_for<0, NM>([&](auto J_) {
        constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
        double dx = 0.0, dy = 0.0;
        static_for<0, n1>([&](auto E_) {
          constexpr int q = decltype(E_)::value;
          if constexpr (q > ex && (q - ex) % 2 == 1 && q + ey <= K) dx = fma(y[0][mode_index<2>(q, ey, 0)], L.dc[q][ex], dx);
          if constexpr (q > ey && (q - ey) % 2 == 1 && q + ex <= K) dy = fma(y[0][mode_index<2>(ex, q, 0)], L.dc[q][ey], dy);
        });
        sd[((v * 2 + 0) * NM + j) * 64 + lane] = dx;
        sd[((v * 2 + 1) * NM + j) * 64 + lane] = dy;
      });
    }
    double mu[4][N];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int l = 0; l < N; ++l) mu[v][l] = 0.0;
    const Line<K> &T = line_const<K>();
#pragma unroll 1
    for (int r = 0; r < n1; ++r) {
      asm volatile("" ::: "memory");  // the LDS rows are read here, not held in registers
      double p[n1];
#pragma unroll
      for (int q = 0; q < n1; ++q) p[q] = T.p[r][q];
      const double wy = T.w[r];
      double U[4][n1], X[4][n1], Y[4][n1];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double c[n1], cx[K], cy[K];
        static_for<0, n1>([&](auto E_) {
          constexpr int ex = decltype(E_)::value;
          double t = sv[(v * N + mode_index<2>(ex, 0, 0)) * 64 + lane];
          static_for<1, n1 - ex>([&](auto Q_) {
            constexpr int q = decltype(Q_)::value;
            t = fma(sv[(v * N + mode_index<2>(ex, q, 0)) * 64 + lane], p[q], t);
          });
          c[ex] = t;
          if constexpr (ex < K) {
            double a = sd[((v * 2 + 0) * NM + mode_index<2>(ex, 0, 0)) * 64 + lane];
            double b = sd[((v * 2 + 1) * NM + mode_index<2>(ex, 0, 0)) * 64 + lane];
            static_for<1, K - ex>([&](auto Q_) {
              constexpr int q = decltype(Q_)::value;
              a = fma(sd[((v * 2 + 0) * NM + mode_index<2>(ex, q, 0)) * 64 + lane], p[q], a);
              b = fma(sd[((v * 2 + 1) * NM + mode_index<2>(ex, q, 0)) * 64 + lane], p[q], b);
            });
            cx[ex] = wy * a;
            cy[ex] = wy * b;
          }
        });
        line_values<K, K>(c, U[v]);
        line_values<K, K - 1>(cx, X[v]);
        line_values<K, K - 1>(cy, Y[v]);
      }
      DG_FENCE;
#pragma unroll
      for (int i = 0; i < n1; ++i) {
        const double u[4] = {U[0][i], U[1][i], U[2][i], U[3][i]};
        const double x[4] = {X[0][i], X[1][i], X[2][i], X[3][i]}, y[4] = {Y[0][i], Y[1][i], Y[2][i], Y[3][i]};
        double G[4];
        flux_vjp2(u, x, y, g.gamma, G);
#pragma unroll
        for (int v = 0; v < 4; ++v) U[v][i] = G[v];
        DG_FENCE;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s[n1];
        line_moments<K, K>(U[v], s);
        static_for<0, N>([&](auto L_) {
          constexpr int l = decltype(L_)::value, ex = mode_exp<2>(l, 0), ey = mode_exp<2>(l, 1);
          if constexpr (ey == 0) mu[v][l] += s[ex];
          else mu[v][l] = fma(s[ex], p[ey], mu[v][l]);
        });
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int l = 0; l < N; ++l) sv[(v * N + l) * 64 + lane] = mu[v][l];
  } else {
    Cell lo = cell, hi = cell;
    bool gl = false, gh = false;  // ghost of a transmissive wall: the other side's trace, no equation
    if (role == 1) {
      lo = row + (Cell)8 * (Cell)(px > 0 ? px - 1 : g.nx - 1);
      gl = g.wall[0] && px == 0;
      gh = g.wall[0] && px == g.nx;
    } else if (role == 2) {
      lo = iy > 0 ? cell - nx8 : cell + (Cell)(g.ny - 1) * nx8;
      gl = g.wall[1] && iy == 0;
    } else {
      hi = iy < g.ny - 1 ? cell + nx8 : cell - (Cell)(g.ny - 1) * nx8;
      gh = g.wall[1] && iy == g.ny - 1;
    }
    // the traces' coefficients in registers, the cotangent's in this wave's
    // place of sm until its moments replace them; one point at a time (a sweep
    // holds about 60 values)
    const int slot = role == 1 ? 0 : role;
    auto cot = [&](int v, int j) __attribute__((always_inline)) -> double & {
      return sm[((slot * 4 + v) * n1 + j) * 64 + lane];
    };
    auto face = [&](auto A_) __attribute__((always_inline)) {
      constexpr int A = decltype(A_)::value;
      double cl[4][n1], ch[4][n1];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double a[1][N], b[1][N], x[1][N], y[1][N], xl[n1], xh[n1];
        load_cell<1, N>(ws, lo, a, (Off)(v * N) * ws.plane);
        load_cell<1, N>(ws, hi, b, (Off)(v * N) * ws.plane);
        load_cell<1, N>(ls, lo, x, (Off)(v * N) * ls.plane);
        load_cell<1, N>(ls, hi, y, (Off)(v * N) * ls.plane);
        edge_coefs<K, A, 1>(a[0], cl[v]);
        edge_coefs<K, A, 0>(b[0], ch[v]);
        edge_coefs<K, A, 1>(x[0], xl);
        edge_coefs<K, A, 0>(y[0], xh);
#pragma unroll
        for (int j = 0; j < n1; ++j) {
          const double s = cl[v][j], t = ch[v][j];
          cl[v][j] = gl ? t : s;
          ch[v][j] = gh ? s : t;
          cot(v, j) = (gh ? 0.0 : xh[j]) - (gl ? 0.0 : xl[j]);
        }
        if (v % 2) DG_FENCE;
      }
      // x: both cells' moments, the lane below's in LDS; y: this cell's alone
      double mo[4][n1];
      auto low = [&](int v, int j) __attribute__((always_inline)) -> double & {
        return sm[((1 * 4 + v) * n1 + j) * 64 + lane];
      };
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < n1; ++j) {
          mo[v][j] = 0.0;
          if (A == 0) low(v, j) = 0.0;
        }
      const Line<K> &T = line_const<K>();
#pragma unroll 1
      for (int i = 0; i < n1; ++i) {
        double p[n1], UL[4], UR[4], G[4], gL[4], gR[4];
#pragma unroll
        for (int j = 0; j < n1; ++j) p[j] = T.p[i][j];
        const double wi = T.w[i];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double a = cl[v][0], b = ch[v][0], c = cot(v, 0);
#pragma unroll
          for (int j = 1; j < n1; ++j) {
            a = fma(cl[v][j], p[j], a);
            b = fma(ch[v][j], p[j], b);
            c = fma(cot(v, j), p[j], c);
          }
          UL[v] = a;
          UR[v] = b;
          G[v] = wi * c;
        }
        hllc_line_vjp<2, A, FX>(UL, UR, g.gamma, G, gL, gR);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          // a ghost's trace is the cell's own
          const double a = gL[v] + (gh ? gR[v] : 0.0), b = gR[v] + (gl ? gL[v] : 0.0);
          const double o = A == 0 || role == 2 ? b : a;
          mo[v][0] += o;
#pragma unroll
          for (int j = 1; j < n1; ++j) mo[v][j] = fma(o, p[j], mo[v][j]);
          if constexpr (A == 0) {
            low(v, 0) += a;
#pragma unroll
            for (int j = 1; j < n1; ++j) low(v, j) = fma(a, p[j], low(v, j));
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < n1; ++j) cot(v, j) = mo[v][j];
    };
    if (role == 1) face(std::integral_constant<int, 0>{});
    else face(std::integral_constant<int, 1>{});
  }
  // variable `role`'s lambda and accumulated gradient, in flight across the barrier
  double lv[N], av[N];
  const Buf as(acc_in ? acc_in : lam, g.nc, 4 * N);
#pragma unroll
  for (int l = 0; l < N; ++l) {
    lv[l] = ls.load(cell, (Off)(role * N + l) * ls.plane);
    av[l] = as.load(cell, (Off)(role * N + l) * ls.plane);
  }
  __syncthreads();

  double mu[N];
#pragma unroll
  for (int l = 0; l < N; ++l) mu[l] = sv[(role * N + l) * 64 + lane];
  auto add = [&](auto A_, auto S_, int q, int at) __attribute__((always_inline)) {
    double m[n1];
#pragma unroll
    for (int j = 0; j < n1; ++j) m[j] = sm[((q * 4 + role) * n1 + j) * 64 + at];
    edge_coefs_t<K, decltype(A_)::value, decltype(S_)::value>(m, mu);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  add(I0{}, I0{}, 0, lane);
  add(I0{}, I1{}, 1, min(lane + 1, 63));
  add(I1{}, I0{}, 2, lane);
  add(I1{}, I1{}, 3, lane);
  if (!own) return;
  const double dt = mode == 0 ? 0.0 : *dtp;
  const Buf os(out, g.nc, 4 * N);
  bool bad = false;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    const Off off = (Off)(role * N + l) * os.plane;
    const double m = g.fac * mu[l];
    bad |= m != m;
    if (mode == 0) {
      os.store(m, cell, off);
    } else if (mode == 1) {
      os.store(av[l] + fma(dt, m, lv[l]), cell, off);
    } else {
      os.store(cb * fma(dt, m, lv[l]), cell, off);
      Buf(acc_out, g.nc, 4 * N).store(mode == 3 ? ca * lv[l] : fma(ca, lv[l], av[l]), cell, off);
    }
  }
  if (bad) atomicOr(flag, FLAG_NAN);
}

}  // namespace dg

int dg::launch_adjoint2d(const dg_ctx *c, const double *w, const double *lam, const double *acc, double *out,
                         double *acc_out, const double *dt, int mode, double ca, double cb, hipStream_t s) {
  AdjointGrid g;
  g.nx = (int)c->nx;
  g.ny = (int)c->ny;
  g.nc = c->ncell;
  for (int a = 0; a < 2; ++a) g.wall[a] = c->cfg.bc[a] == DG_BC_TRANSMISSIVE;
  g.fac = 2.0 / c->dx / 4.0;
  g.gamma = c->cfg.gamma;
  g.columns = (long)(g.nx + 1) * g.ny;
  const dim3 nb((unsigned)((g.columns + 62) / 63));
  auto go = [&](auto K_) {
    constexpr int K = decltype(K_)::value;
    // byte offsets of 32 bits in the state (below 4 GB), else in each plane
    // (below 2^29 cells), else of 64 bits (from k = 2 on three such states do
    // not fit the card)
    auto pick = [&](auto B_) {
      using Buf = std::remove_pointer_t<decltype(B_)>;
      return c->cfg.flux == DG_HLLC_DAVIS ? k_adjoint_split2d<K, DG_HLLC_DAVIS, Buf> : k_adjoint_split2d<K, DG_HLLC_BATTEN, Buf>;
    };
    auto kernel = pick((StateBuf *)nullptr);
    if (c->ncell * 8LL * c->sh.nv * c->sh.N >= (1LL << 32)) kernel = pick((StatePlanes *)nullptr);
    if (c->ncell >= (1L << 29)) {
      if constexpr (K > 1) return (int)hipErrorOutOfMemory;
      else kernel = pick((StatePtr *)nullptr);
    }
    hipLaunchKernelGGL(kernel, nb, dim3(256), 0, s, w, lam, acc, out, acc_out, dt, g, mode, ca, cb, c->flag);
    return (int)hipGetLastError();
  };
  if (c->sh.k == 1) return go(std::integral_constant<int, 1>{});
  if (c->sh.k == 2) return go(std::integral_constant<int, 2>{});
  return go(std::integral_constant<int, 3>{});
}
