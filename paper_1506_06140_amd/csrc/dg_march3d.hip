// 3D right-hand side + stage, one thread per cell, sum-factorised (FP64).
#include "dg_march.h"
#include "dg_rules.h"

namespace dg {

struct MarchGrid {
  int nx, ny, nz;
  long nc;
  int wall[3];      // transmissive walls along each axis
  double fac;       // (2/dx) 2^-d
  double gamma;
  int len;          // planes a wave marches through
  long columns;     // (nx + 2) ny ceil(nz / len)
};

// Volume integral (eq. dg_term2) of one cell, added to acc: the state at the
// Gauss nodes one axis at a time, the nine distinct non-trivial fluxes there
// (the momentum flux tensor is symmetric), and their moments against the
// polynomials of degree <= K - 1, which hold the basis gradients
// (P~_e' = sum_j dc_ej P~_j).  The mass flux is the momentum, a polynomial of
// the cell, so its moments are 2^3 times the momentum's own weights (the rule
// integrates their products exactly).
// The result starts from the lower z face's moments m and goes to set(v, row).
template <int K, class W, class Set>
__device__ __forceinline__ void volume_term(W &&w, double gm1, const double (&m)[5][(K + 1) * (K + 2) / 2], Set &&set) {
  constexpr int n1 = K + 1, N = (K + 1) * (K + 2) * (K + 3) / 6, N2 = (K + 1) * (K + 2) / 2;
  constexpr int NM = K * (K + 1) * (K + 2) / 6;
  constexpr Line<K> L{};
  const Line<K> &T = line_const<K>();
  double M[9][NM];  // xx xy xz yy yz zz, hx hy hz
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < NM; ++j) M[t][j] = 0.0;
#pragma unroll 1
  for (int iz = 0; iz < n1; ++iz) {
    double pz[n1];
#pragma unroll
    for (int e = 0; e < n1; ++e) pz[e] = T.p[iz][e];
    const double wz = T.w[iz];
    double c2[5][N2];
#pragma unroll
    for (int v = 0; v < 5; ++v)
      static_for<0, N2>([&](auto J_) {
        constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
        double t = w(v, mode_index<3>(ex, ey, 0));
        static_for<1, n1 - ex - ey>([&](auto G_) {
          constexpr int ez = decltype(G_)::value;
          t = fma(w(v, mode_index<3>(ex, ey, ez)), pz[ez], t);
        });
        c2[v][j] = t;
      });
    DG_FENCE;
#pragma unroll
    for (int iy = 0; iy < n1; ++iy) {
      double U[5][n1];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        double c1[n1];
        static_for<0, n1>([&](auto E_) {
          constexpr int ex = decltype(E_)::value;
          double t = c2[v][mode_index<2>(ex, 0, 0)];
          static_for<1, n1 - ex>([&](auto G_) {
            constexpr int ey = decltype(G_)::value;
            t = L.p[iy][ey] == 0.0 ? t : fma(c2[v][mode_index<2>(ex, ey, 0)], L.p[iy][ey], t);
          });
          c1[ex] = t;
        });
        line_values<K, K>(c1, U[v]);
      }
      double G[9][n1];
#pragma unroll
      for (int i = 0; i < n1; ++i) {
        const double ir = rcp3(U[0][i]);
        const double vx = U[1][i] * ir, vy = U[2][i] * ir, vz = U[3][i] * ir;
        const double ke = fma(U[1][i], vx, fma(U[2][i], vy, U[3][i] * vz));
        const double p = gm1 * fma(-0.5, ke, U[4][i]), H = U[4][i] + p;
        G[0][i] = fma(U[1][i], vx, p);
        G[1][i] = U[1][i] * vy;
        G[2][i] = U[1][i] * vz;
        G[3][i] = fma(U[2][i], vy, p);
        G[4][i] = U[2][i] * vz;
        G[5][i] = fma(U[3][i], vz, p);
        G[6][i] = H * vx;
        G[7][i] = H * vy;
        G[8][i] = H * vz;
      }
      DG_FENCE;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        double s[K];
        line_moments<K, K - 1>(G[t], s);
        static_for<0, NM>([&](auto J_) {
          constexpr int j = decltype(J_)::value, ex = mode_exp<3>(j, 0), ey = mode_exp<3>(j, 1), ez = mode_exp<3>(j, 2);
          if (L.p[iy][ey] != 0.0) M[t][j] = fma(s[ex], (L.w[iy] * L.p[iy][ey]) * (wz * pz[ez]), M[t][j]);
        });
      }
      DG_FENCE;
    }
  }
  // V_l = sum_a sum_j dc[e_a][j] M_a[e with e_a -> j]
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double acc[N];
#pragma unroll
    for (int l = 0; l < N; ++l) acc[l] = 0.0;
    face_lift<K, 2, 0>(m[v], acc);
    static_for<1, N>([&](auto L_) {
      constexpr int l = decltype(L_)::value, ex = mode_exp<3>(l, 0), ey = mode_exp<3>(l, 1), ez = mode_exp<3>(l, 2);
      static_for<0, 3>([&](auto A_) {
        constexpr int a = decltype(A_)::value, ea = a == 0 ? ex : a == 1 ? ey : ez;
        static_for<0, ea>([&](auto J_) {
          constexpr int j = decltype(J_)::value;
          if constexpr ((ea - j) % 2 == 1) {
            constexpr int q = a == 0 ? mode_index<3>(j, ey, ez) : a == 1 ? mode_index<3>(ex, j, ez) : mode_index<3>(ex, ey, j);
            constexpr double dc = L.dc[ea][j];
            const int t = v == 1 ? a : v == 2 ? (a == 0 ? 1 : a == 1 ? 3 : 4) : v == 3 ? (a == 0 ? 2 : a == 1 ? 4 : 5) : 6 + a;
            acc[l] = v == 0 ? fma(w(1 + a, q), 8.0 * dc, acc[l]) : fma(M[t][q], dc, acc[l]);
          }
        });
      });
    });
    set(v, acc);
    DG_FENCE;
  }
}

// 3D right-hand side and stage, one thread per cell.
//
// FP64 matrix and vector instructions share one datapath, so what counts is
// the number of operations: contracted one axis at a time (the basis is a
// total-degree set of products of 1D polynomials) a cell at k = 2 takes about
// a sixth of the multiply-adds of the dense tables, and the Riemann solver,
// about 165 issue slots per face point, is what is left.  So most faces are
// solved once:
//   x  a wave holds 64 consecutive positions of rows extended by one halo
//      cell at each end; a lane solves the face to the lane below it (whose
//      trace arrives by a DPP shift) and hands the flux's moments down; lanes
//      1..62 are real, so rows of any length fill the waves;
//   z  the wave marches along z, the upper face's moments of one cell being
//      the lower face's of the next;
//   y  is solved by both cells from the same coefficients with the same code,
//      so both obtain the same flux bit for bit.
// One wave per SIMD at k = 2 (450 registers: the own cell 100, a face's
// coefficients and moments 120, the next neighbour in flight 100), two at
// k = 1; the accumulators and the low side's trace sit in LDS (40 KB a wave,
// lane-private, no barrier).  A first form with everything in registers
// spilled 90 of them and spent 64 % of its cycles waiting on scratch and
// loads (128^3, k = 2: 3240 us).  128^3, one launch: k = 2 2708 us (MFMA
// kernel) -> 1346 us, VALU issuing 63 % and all units 77 % of the cycles;
// k = 1 681 us (k_rhs_stage) -> 441 us, VALU 85 %.
template <int K, int FX, bool PER>
__global__ __launch_bounds__(64, 1) void k_rhs_march3d(const double *__restrict__ w, double *__restrict__ out,
                                                       const double *__restrict__ dtp, MarchGrid g, int mode, Mix mx,
                                                       int *__restrict__ flag) {
  constexpr int N = (K + 1) * (K + 2) * (K + 3) / 6, N2 = (K + 1) * (K + 2) / 2;
  __shared__ double sa[5 * N * 64];   // this lane's accumulators V - S: [v][l][lane]
  __shared__ double sx[5 * N2 * 64];  // trace coefficients of a face's low side: [v][j][lane]
  const int lane = threadIdx.x;
  // XCD b mod 8 takes a contiguous band of the columns
  const int nb = gridDim.x, xcd = blockIdx.x % 8, jb = blockIdx.x / 8;
  const long blk = (long)xcd * (nb / 8) + min(xcd, nb % 8) + jb;
  const long e0 = 62 * blk + lane - 1;
  const long e = min(max(e0, 0L), g.columns - 1);
  const unsigned px = (unsigned)(e % (g.nx + 2)), rest = (unsigned)(e / (g.nx + 2));
  const int iy = (int)(rest % (unsigned)g.ny), z0 = (int)(rest / (unsigned)g.ny) * g.len;
  int ix = (int)px - 1;
  const bool own = ix >= 0 && ix < g.nx && lane > 0 && lane < 63 && e0 < g.columns;
  // ghost selects of the face between this lane and the lane below it
  const bool ghost_l = !PER && g.wall[0] && px == 1, ghost_r = !PER && g.wall[0] && px == (unsigned)g.nx + 1;
  if (ix < 0) ix = g.nx - 1;
  if (ix >= g.nx) ix = 0;
  // byte offsets within a plane of the state
  const StateBuf ws(w, g.nc, 5 * N), os(out, g.nc, 5 * N);
  const StateBuf ys(mode != 0 && mx.n > 0 ? mx.y[0] : w, g.nc, 5 * N);
  const unsigned nxy8 = 8u * (unsigned)g.nx * (unsigned)g.ny, nx8 = 8u * (unsigned)g.nx;
  const unsigned col = 8u * ((unsigned)iy * (unsigned)g.nx + (unsigned)ix);
  const bool wyl = !PER && g.wall[1] && iy == 0, wyh = !PER && g.wall[1] && iy == g.ny - 1;
  const unsigned dyl = iy > 0 ? 0u - nx8 : (wyl ? 0u : nxy8 - nx8), dyh = iy < g.ny - 1 ? nx8 : (wyh ? 0u : nx8 - nxy8);
  const double gm1 = g.gamma - 1.0;
  // out = scale (V - S) + cu w + sum a_k y_k (mode 0: no extra terms)
  const double scale = mode == 0 ? g.fac : g.fac * (mx.cl * *dtp), cu = mode == 0 ? 0.0 : mx.cu;
  const int ny0 = mode == 0 ? 0 : mx.n;
  bool bad = false;
  auto low = [&](int v, int j) __attribute__((always_inline)) -> double & { return sx[(v * N2 + j) * 64 + lane]; };
  auto acc_row = [&](int v, double (&r)[N]) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < N; ++l) r[l] = sa[(v * N + l) * 64 + lane];
  };
  auto set_acc = [&](int v, const double (&r)[N]) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < N; ++l) sa[(v * N + l) * 64 + lane] = r[l];
  };
  auto plane = [&](int zr) {  // the plane of z index zr, wrapped or held at a wall
    const int zl = !PER && g.wall[2] ? 0 : g.nz - 1, zh = (!PER && g.wall[2]) || zr > g.nz ? g.nz - 1 : 0;
    return (unsigned)(zr < 0 ? zl : zr < g.nz ? zr : zh) * nxy8;
  };

  double wc[5][N];  // this lane's own cell
  load_cell<5, N>(ws, plane(z0 - 1) + col, wc);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double t[N2];
    face_coefs<K, 2, 1>(wc[v], t);
#pragma unroll
    for (int j = 0; j < N2; ++j) low(v, j) = t[j];
  }
  load_cell<5, N>(ws, plane(z0) + col, wc);
#pragma unroll 1
  for (int s = 0; s <= g.len; ++s) {
    const int zr = z0 + s;  // the cell above the face
    const unsigned cell = plane(zr) + col;
    double m[5][N2], ch[5][N2];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      face_coefs<K, 2, 0>(wc[v], ch[v]);
      if constexpr (!PER) {
        const bool gl = g.wall[2] && zr == 0, gh = g.wall[2] && zr >= g.nz;
#pragma unroll
        for (int j = 0; j < N2; ++j) {
          const double x = low(v, j), y = ch[v][j];
          low(v, j) = gl ? y : x;
          ch[v][j] = gh ? x : y;
        }
      }
    }
    DG_FENCE;
    const bool st = own && s > 0 && zr - 1 < g.nz;
    const unsigned cb = (unsigned)min(max(zr - 1, 0), g.nz - 1) * nxy8 + col;
    double y0[5][N];
    load_cell<5, N, NT>(ys, cb, y0);  // in flight during the face
    DG_FENCE;
    face_flux<K, 2, FX>(low, ch, g.gamma, m);
    if (s > 0) {  // the cell below is complete: its last face and its stage update
      unsigned off = 0;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        double sm[N2], a[N];
#pragma unroll
        for (int j = 0; j < N2; ++j) {
          sm[j] = scale * m[v][j];
          bad |= st && m[v][j] != m[v][j];
        }
        acc_row(v, a);
        face_lift<K, 2, 1>(sm, a);
#pragma unroll
        for (int l = 0; l < N; ++l) {
          a[l] = ny0 > 0 ? fma(mx.a[0], y0[v][l], a[l]) : a[l];
          if (ny0 > 1 && st) a[l] = mix_tail(mx, a[l], (long)(v * N + l) * g.nc + (cb >> 3), 1);
          if (st) os.store<NT>(a[l], cb, off);
          off += os.plane;
        }
        DG_FENCE;
      }
    }
    if (s == g.len) break;
    volume_term<K>([&](int v, int l) __attribute__((always_inline)) { return wc[v][l]; }, gm1, m, set_acc);
    DG_FENCE;
    // x faces: each lane the face to the lane below it
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double h[N2];
      face_coefs<K, 0, 1>(wc[v], h);
      face_coefs<K, 0, 0>(wc[v], ch[v]);
#pragma unroll
      for (int j = 0; j < N2; ++j) {
        const double b = lane_below(h[j]), o = ch[v][j];
        low(v, j) = ghost_l ? o : b;
        if constexpr (!PER) ch[v][j] = ghost_r ? b : o;
      }
      DG_FENCE;
    }
    double nb[5][N];
    load_cell<5, N>(ws, cell + dyl, nb);  // in flight during the face
    DG_FENCE;
    face_flux<K, 0, FX>(low, ch, g.gamma, m);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double a[N];
      acc_row(v, a);
      face_lift<K, 0, 0>(m[v], a);
#pragma unroll
      for (int j = 0; j < N2; ++j) m[v][j] = lane_above(m[v][j]);
      face_lift<K, 0, 1>(m[v], a);
      set_acc(v, a);
      DG_FENCE;
    }
    auto y_side = [&](auto S_, bool wy, unsigned next) __attribute__((always_inline)) {
      constexpr int S = decltype(S_)::value;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        double c[N2], o[N2];
        face_coefs<K, 1, 1 - S>(nb[v], c);
        face_coefs<K, 1, S>(wc[v], o);
#pragma unroll
        for (int j = 0; j < N2; ++j) {
          const double n = !PER && wy ? o[j] : c[j];
          low(v, j) = S == 0 ? n : o[j];
          ch[v][j] = S == 0 ? o[j] : n;
        }
        DG_FENCE;
      }
      load_cell<5, N>(ws, next, nb);
      DG_FENCE;
      face_flux<K, 1, FX>(low, ch, g.gamma, m);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        double a[N];
        acc_row(v, a);
        face_lift<K, 1, S>(m[v], a);
        if constexpr (S == 1) {  // all but the upper face: scaled, with the cell's own term
#pragma unroll
          for (int l = 0; l < N; ++l) {
            bad |= own && zr < g.nz && a[l] != a[l];
            a[l] *= scale;
            if (mode != 0) a[l] = fma(cu, wc[v][l], a[l]);
          }
        }
        set_acc(v, a);
        DG_FENCE;
      }
    };
    y_side(std::integral_constant<int, 0>{}, wyl, cell + dyh);
    y_side(std::integral_constant<int, 1>{}, wyh, plane(zr + 1) + col);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double t[N2];
      face_coefs<K, 2, 1>(wc[v], t);
#pragma unroll
      for (int j = 0; j < N2; ++j) low(v, j) = t[j];
    }
    DG_FENCE;
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int l = 0; l < N; ++l) wc[v][l] = nb[v][l];
  }
  if (bad) atomicOr(flag, FLAG_NAN);
}

}  // namespace dg

// FP64 on uniform 3D grids at k = 1 and 2 without gravity, states below 4 GB
// (32-bit byte offsets), of the sizes where it is faster.
bool dg::march3d_takes(const dg_ctx *c) {
  if (c->sh.d != 3 || c->sh.k > 2 || c->amr || c->gravity || c->tree) return false;
  if (c->cfg.precision != DG_FP64 || c->cfg.path3d != DG_PATH3D_AUTO) return false;
  if (c->ncell * 8 * c->sh.nv * c->sh.N >= (1LL << 32)) return false;
  return march3d_faster(c->sh.k, c->nx, c->ny, c->nz);
}

int dg::launch_march3d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                       hipStream_t s) {
  MarchGrid g;
  g.nx = (int)c->nx;
  g.ny = (int)c->ny;
  g.nz = (int)c->nz;
  g.nc = c->ncell;
  bool per = true;
  for (int a = 0; a < 3; ++a) {
    g.wall[a] = c->cfg.bc[a] == DG_BC_TRANSMISSIVE;
    per = per && !g.wall[a];
  }
  g.fac = 2.0 / c->dx / 8.0;
  g.gamma = c->cfg.gamma;
  const long row = (long)(g.nx + 2) * g.ny;
  g.len = march_len(row, g.nz, march_slots(c->sh.k));
  g.columns = row * ((g.nz + g.len - 1) / g.len);
  const dim3 nb((unsigned)((g.columns + 61) / 62));
  auto go = [&](auto K_, auto FX_) {
    constexpr int K = decltype(K_)::value, FX = decltype(FX_)::value;
    if (per)
      hipLaunchKernelGGL((k_rhs_march3d<K, FX, true>), nb, dim3(64), 0, s, w, out, dt, g, mode, mx, c->flag);
    else
      hipLaunchKernelGGL((k_rhs_march3d<K, FX, false>), nb, dim3(64), 0, s, w, out, dt, g, mode, mx, c->flag);
  };
  using B = std::integral_constant<int, DG_HLLC_BATTEN>;
  using V = std::integral_constant<int, DG_HLLC_DAVIS>;
  const bool dav = c->cfg.flux == DG_HLLC_DAVIS;
  if (c->sh.k == 1) dav ? go(std::integral_constant<int, 1>{}, V{}) : go(std::integral_constant<int, 1>{}, B{});
  else dav ? go(std::integral_constant<int, 2>{}, V{}) : go(std::integral_constant<int, 2>{}, B{});
  return (int)hipGetLastError();
}
