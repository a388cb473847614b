// 2D right-hand side + stage, a cell's work split over four waves (FP64).
#include "dg_march.h"
#include "dg_rules.h"

#include <algorithm>

namespace dg {

// moments m[v][e] of the HLLC flux over the K + 1 face points, two points'
// solves interleaved (PAIR) or one at a time
template <int K, int A, int FX, bool PAIR>
__device__ __forceinline__ void edge_flux(const double (&cl)[4][K + 1], const double (&ch)[4][K + 1], double gamma,
                                          double (&m)[4][K + 1]) {
  constexpr int n1 = K + 1;
  double ul[4][n1], uh[4][n1];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    line_values<K, K>(cl[v], ul[v]);
    line_values<K, K>(ch[v], uh[v]);
  }
  DG_FENCE;
  double F[4][n1];
#pragma unroll
  for (int i = 0; i < n1; ++i) {
    const double UL[4] = {ul[0][i], ul[1][i], ul[2][i], ul[3][i]}, UR[4] = {uh[0][i], uh[1][i], uh[2][i], uh[3][i]};
    double f[4];
    hllc_line<2, A, FX>(UL, UR, gamma, f);
#pragma unroll
    for (int v = 0; v < 4; ++v) F[v][i] = f[v];
    if (!PAIR || i % 2 == 1) DG_FENCE;
  }
  DG_FENCE;
#pragma unroll
  for (int v = 0; v < 4; ++v) line_moments<K, K>(F[v], m[v]);
}

// the outward flux of side S (moments m) taken off the accumulators
template <int K, int A, int S>
__device__ __forceinline__ void edge_lift(const double (&m)[K + 1], double (&acc)[(K + 1) * (K + 2) / 2]) {
  constexpr Line<K> L{};
  static_for<0, (K + 1) * (K + 2) / 2>([&](auto L_) {
    constexpr int l = decltype(L_)::value, ex = mode_exp<2>(l, 0), ey = mode_exp<2>(l, 1);
    constexpr int n = A == 0 ? ex : ey, t = A == 0 ? ey : ex;
    constexpr double s = (S == 0 ? (n % 2 ? -1.0 : 1.0) : -1.0) * L.b[n];
    acc[l] = fma(m[t], s, acc[l]);
  });
}

// Volume integral of one cell (see volume_term in dg_march3d.hip), with the
// gravity source (GRAV: its values at the nodes, (dx/2) w_q included, through
// gv(axis, node)), variable by variable through set(v, row).
template <int K, bool GRAV, class W, class G2, class Set>
__device__ __forceinline__ void area_term(W &&w, double gm1, G2 &&gv, Set &&set) {
  constexpr int n1 = K + 1, N = (K + 1) * (K + 2) / 2, NM = K * (K + 1) / 2;
  constexpr Line<K> L{};
  const Line<K> &T = line_const<K>();
  double M[5][NM];  // xx xy yy, hx hy
  double src[3][GRAV ? N : 1];  // the source's projection (momenta, energy)
  if constexpr (GRAV)
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int l = 0; l < N; ++l) src[t][l] = 0.0;
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int j = 0; j < NM; ++j) M[t][j] = 0.0;
#pragma unroll 1
  for (int iy = 0; iy < n1; ++iy) {
    asm volatile("" ::: "memory");  // weights in LDS are read row by row, not held in registers
    double p[n1];
#pragma unroll
    for (int e = 0; e < n1; ++e) p[e] = T.p[iy][e];
    const double wy = T.w[iy];
    double U[4][n1];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double c1[n1];
      static_for<0, n1>([&](auto E_) {
        constexpr int ex = decltype(E_)::value;
        double t = w(v, mode_index<2>(ex, 0, 0));
        static_for<1, n1 - ex>([&](auto Y_) {
          constexpr int ey = decltype(Y_)::value;
          t = fma(w(v, mode_index<2>(ex, ey, 0)), p[ey], t);
        });
        c1[ex] = t;
      });
      line_values<K, K>(c1, U[v]);
    }
    double G[5][n1], S[3][n1];
#pragma unroll
    for (int i = 0; i < n1; ++i) {
      const double ir = rcp3(U[0][i]);
      const double vx = U[1][i] * ir, vy = U[2][i] * ir;
      const double ke = fma(U[1][i], vx, U[2][i] * vy);
      const double pr = gm1 * fma(-0.5, ke, U[3][i]), H = U[3][i] + pr;
      G[0][i] = fma(U[1][i], vx, pr);
      G[1][i] = U[1][i] * vy;
      G[2][i] = fma(U[2][i], vy, pr);
      G[3][i] = H * vx;
      G[4][i] = H * vy;
      if constexpr (GRAV) {  // the values carry (dx/2) w_q
        const double gx = gv(0, iy * n1 + i), gy = gv(1, iy * n1 + i);
        S[0][i] = U[0][i] * gx;
        S[1][i] = U[0][i] * gy;
        S[2][i] = fma(U[1][i], gx, U[2][i] * gy);
      }
    }
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      double s[K];
      line_moments<K, K - 1>(G[t], s);
      static_for<0, NM>([&](auto J_) {
        constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
        M[t][j] = fma(s[ex], wy * p[ey], M[t][j]);
      });
    }
    if constexpr (GRAV) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        static_for<0, n1>([&](auto E_) {
          constexpr int ex = decltype(E_)::value;
          double s = S[t][0] * L.p[0][ex];
#pragma unroll
          for (int i = 1; i < n1; ++i) s = fma(S[t][i], L.p[i][ex], s);
          static_for<0, n1 - ex>([&](auto Y_) {
            constexpr int ey = decltype(Y_)::value, l = mode_index<2>(ex, ey, 0);
            src[t][l] = fma(s, p[ey], src[t][l]);
          });
        });
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    double acc[N];
#pragma unroll
    for (int l = 0; l < N; ++l) acc[l] = GRAV && v > 0 ? src[v - 1][l] : 0.0;
    static_for<1, N>([&](auto L_) {
      constexpr int l = decltype(L_)::value, ex = mode_exp<2>(l, 0), ey = mode_exp<2>(l, 1);
      static_for<0, 2>([&](auto A_) {
        constexpr int a = decltype(A_)::value, ea = a == 0 ? ex : ey;
        static_for<0, ea>([&](auto J_) {
          constexpr int j = decltype(J_)::value;
          if constexpr ((ea - j) % 2 == 1) {
            constexpr int q = a == 0 ? mode_index<2>(j, ey, 0) : mode_index<2>(ex, j, 0);
            constexpr double dc = L.dc[ea][j];
            const int t = v == 1 ? a : v == 2 ? 1 + a : 3 + a;
            acc[l] = v == 0 ? fma(w(1 + a, q), 4.0 * dc, acc[l]) : fma(M[t][q], dc, acc[l]);
          }
        });
      });
    });
    set(v, acc);
  }
}

struct SplitGrid {
  int nx, ny;
  long nc;
  int wall[2];
  double fac, gamma;
  long columns;  // (nx + 1) ny
};

// 2D right-hand side and stage.
//
// A block of four waves takes 64 consecutive positions of rows extended by one
// (position nx of a row is only the face behind its last cell; the last lane
// is the next block's first).  Wave 0 forms the cells' volume terms, waves 1,
// 2 and 3 the fluxes of their x low, y low and y high faces; the high x face
// is the next lane's low one.  After one barrier wave v lifts the four faces'
// moments of variable v onto its volume term and applies the stage update.
// Each phase is a contraction of one axis at a time in one lane (no
// reduction over lanes, no table reads), the four phases cost about the same
// (k = 2: 440 issue slots the volume, 520 a face), and a y face is solved by
// both of its cells with the same code and inputs: the same flux bit for bit.
// A small grid is bound by the length of one wave's work, which the split cuts
// to a third of a cell's; a large one by the vector ALU (43 % at 512^2, k = 2)
// and its loads' latency, with the memory floor at half its time.
// Against the 8x8 tiles of four lanes per cell, us per launch: k = 1 32^2 5.6
// -> 4.0, 256^2 10.0 -> 8.5; k = 2 32^2 7.8 -> 5.2, 256^2 17.9 -> 14.3, 512^2 64
// -> 40.5; k = 3 32^2 11.6 -> 7.1, 512^2 127 -> 76; k = 4 32^2 33.6 -> 11.7, 256^2
// 77.5 -> 39.7.  One thread per cell marching along y (no second solve of a y
// face) took 9.4, 19.5 and 46 us at k = 2.  Loading the own cell once per block
// and sharing its traces through LDS halved the loads and changed nothing.
// Registers bound the waves per SIMD below: one step lower spills, and 30
// spilled registers cost 60 % (k = 3, 512^2: 76 -> 124 us).
template <int K, int FX, bool PER, bool GRAV>
__global__ __launch_bounds__(256, GRAV ? (K == 1 ? 4 : K == 2 ? 2 : 1) : K == 1 ? 5 : K == 2 ? 4 : K == 3 ? 3 : 2) void k_rhs_split2d(
    const double *__restrict__ w, double *__restrict__ out, const double *__restrict__ dtp, SplitGrid g, int mode, Mix mx,
    int *__restrict__ flag, RateOp ro, const double *__restrict__ grav) {
  constexpr int N = (K + 1) * (K + 2) / 2, n1 = K + 1;
  __shared__ double sv[4 * N * 64];       // volume term [v][l][lane]
  __shared__ double sm[3 * 4 * n1 * 64];  // face moments [face: x low, y low, y high][v][e][lane]
  __shared__ double mean[4 * 64];
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = gridDim.x, xcd = blockIdx.x % 8, jb = blockIdx.x / 8;
  const long blk = (long)xcd * (nb / 8) + min(xcd, nb % 8) + jb;
  const long e0 = 63 * blk + lane;
  const long e = min(e0, g.columns - 1);
  const int px = (int)((unsigned)e % (unsigned)(g.nx + 1)), iy = (int)((unsigned)e / (unsigned)(g.nx + 1));
  const bool own = px < g.nx && lane < 63 && e0 < g.columns;
  const StateBuf ws(w, g.nc, 4 * N), os(out, g.nc, 4 * N);
  const unsigned nx8 = 8u * (unsigned)g.nx, row = (unsigned)iy * nx8;
  const unsigned cell = row + 8u * (unsigned)(px < g.nx ? px : 0);
  double dt = 0.0;
  if (mode != 0) {
    if (ro.op == RATE_DT) {
      double r = 0.0;
#pragma unroll
      for (int k = 0; k < RATE_SLOTS; ++k)
        r = fmax(r, __longlong_as_double((long long)*rate_slot(ro.word, k)));
      dt = ro.cfl_fk / r;
      if (blockIdx.x == 0 && threadIdx.x == 0) ro.dt_out[0] = dt;
    } else {
      dt = *dtp;
    }
  }
  if (blockIdx.x == 0 && ro.op == RATE_CLEAR && threadIdx.x < RATE_SLOTS) ro.word[RATE_STRIDE * threadIdx.x] = 0ull;

  if (role == 0) {
    double wc[4][N];
    load_cell<4, N>(ws, cell, wc);
    // at k >= 3 the weights wait in LDS (the term's own place: its rows of the
    // momenta are read before they are replaced)
    if constexpr (K >= 3)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int l = 0; l < N; ++l) sv[(v * N + l) * 64 + lane] = wc[v][l];
    area_term<K, GRAV>(
        [&](int v, int l) __attribute__((always_inline)) {
          if constexpr (K >= 3) return sv[(v * N + l) * 64 + lane];
          else return wc[v][l];
        },
        g.gamma - 1.0,
        [&](int a, int q) __attribute__((always_inline)) {
          return GRAV ? grav[(long)(a * n1 * n1 + q) * g.nc + (cell >> 3)] : 0.0;
        },
        [&](int v, const double(&row)[N]) __attribute__((always_inline)) {
#pragma unroll
          for (int l = GRAV ? 0 : 1; l < N; ++l) sv[(v * N + l) * 64 + lane] = row[l];
        });
  } else {
    // the face's two cells; a ghost (transmissive wall) takes the other's trace
    unsigned lo = cell, hi = cell;
    bool gl = false, gh = false;
    if (role == 1) {
      lo = row + 8u * (unsigned)(px > 0 ? px - 1 : g.nx - 1);
      if constexpr (!PER) {
        gl = g.wall[0] && px == 0;
        gh = g.wall[0] && px == g.nx;
      }
    } else if (role == 2) {
      lo = iy > 0 ? cell - nx8 : cell + (unsigned)(g.ny - 1) * nx8;
      if constexpr (!PER) gl = g.wall[1] && iy == 0;
    } else {
      hi = iy < g.ny - 1 ? cell + nx8 : cell - (unsigned)(g.ny - 1) * nx8;
      if constexpr (!PER) gh = g.wall[1] && iy == g.ny - 1;
    }
    double cl[4][n1], ch[4][n1], m[4][n1];
    auto face = [&](auto A_) __attribute__((always_inline)) {
      constexpr int A = decltype(A_)::value;
      // two variables' weights at a time at k >= 3: all eight rows at once
      // would be the kernel's register peak
#pragma unroll
      for (int v0 = 0; v0 < 4; v0 += (K >= 3 ? 2 : 4)) {
        constexpr int NVL = K >= 3 ? 2 : 4;
        double a[NVL][N], b[NVL][N];
        const unsigned off = (unsigned)(v0 * N) * ws.plane;
        load_cell<NVL, N>(ws, lo, a, off);
        load_cell<NVL, N>(ws, hi, b, off);
#pragma unroll
        for (int i = 0; i < NVL; ++i) {
          const int v = v0 + i;
          edge_coefs<K, A, 1>(a[i], cl[v]);
          edge_coefs<K, A, 0>(b[i], ch[v]);
          if constexpr (!PER)
#pragma unroll
            for (int j = 0; j < n1; ++j) {
              const double x = cl[v][j], y = ch[v][j];
              cl[v][j] = gl ? y : x;
              ch[v][j] = gh ? x : y;
            }
        }
        if constexpr (K >= 3) DG_FENCE;
      }
      // with walls at k = 2 a pair of solves spills four registers (256^2: 15.3
      // us against 14.1; without walls a pair takes 13.7, single ones 14.4)
      edge_flux<K, A, FX, PER || K != 2>(cl, ch, g.gamma, m);
    };
    if (role == 1) face(std::integral_constant<int, 0>{});
    else face(std::integral_constant<int, 1>{});
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < n1; ++j) sm[(((role - 1) * 4 + v) * n1 + j) * 64 + lane] = m[v][j];
  }
  // the operands of this wave's share of the update (variable `role`), in
  // flight across the barrier
  double wo[N], y0[N];
  const StateBuf ys(mode != 0 && mx.n > 0 ? mx.y[0] : w, g.nc, 4 * N);
#pragma unroll
  for (int l = 0; l < N; ++l) {
    wo[l] = ws.load(cell, (unsigned)(role * N + l) * ws.plane);
    y0[l] = ys.load(cell, (unsigned)(role * N + l) * ws.plane);
  }
  __syncthreads();

  // variable `role`: the four faces lifted onto the volume term, the update
  double acc[N];
  acc[0] = GRAV ? sv[role * N * 64 + lane] : 0.0;
#pragma unroll
  for (int l = 1; l < N; ++l) acc[l] = sv[(role * N + l) * 64 + lane];
  auto moments = [&](int f, int at, double (&m)[n1]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < n1; ++j) m[j] = sm[((f * 4 + role) * n1 + j) * 64 + at];
  };
  double m[n1];
  moments(0, lane, m);
  edge_lift<K, 0, 0>(m, acc);
  moments(0, min(lane + 1, 63), m);
  edge_lift<K, 0, 1>(m, acc);
  moments(1, lane, m);
  edge_lift<K, 1, 0>(m, acc);
  moments(2, lane, m);
  edge_lift<K, 1, 1>(m, acc);
  bool bad = false;
  const double cldt = mx.cl * dt;
  if (own) {
    unsigned off = (unsigned)(role * N) * os.plane;
#pragma unroll
    for (int l = 0; l < N; ++l) {
      const double L = g.fac * acc[l];
      bad |= L != L;
      double o = L;
      if (mode != 0) {
        o = fma(cldt, L, mx.cu * wo[l]);
        if (mx.n > 0) o = fma(mx.a[0], y0[l], o);
        if (mx.n > 1) o = mix_tail(mx, o, (long)(role * N + l) * g.nc + (cell >> 3), 1);
      }
      os.store(o, cell, off);
      off += os.plane;
      if (l == 0) mean[role * 64 + lane] = o;
    }
  }
  if (bad) atomicOr(flag, FLAG_NAN);
  if (ro.op == RATE_FOLD) {
    // signal rate of the new means (the limiters leave them unchanged): a wave
    // max, one global max per block
    __syncthreads();
    if (role == 0) {
      double r = 0.0;
      if (own) {
        const double U[4] = {mean[lane], mean[64 + lane], mean[128 + lane], mean[192 + lane]};
        bool neg = false;
        r = cell_rate<2>(U, g.gamma, ro.dx, neg, ro.gk, ro.gmax ? ro.gmax[cell >> 3] : 0.0);
        if (neg) atomicOr(flag, FLAG_NEGATIVE);
      }
      r = wave_max(r);
      if (lane == 0) atomicMax(rate_slot(ro.word, blockIdx.x), (unsigned long long)__double_as_longlong(r));
    }
  }
}

// Quadtree right-hand side and stage: five waves per 64 leaves, the volume
// term and the fluxes of the four sides (both leaves of a face solve it, with
// the same code and inputs), then one variable per wave as above.  A side is
// one face (same level, wall), two half faces (finer neighbours: this leaf's
// trace at the mapped nodes (eta + sigma)/2, the moments weighted w_r / 2) or
// one face against a coarser neighbour (its trace at this leaf's half), so
// each lane reads the values of P~_e at its own and its neighbour's nodes from
// one of three tables in LDS.  Bound by the length of a wave's work (17 000
// leaves are 270 blocks): the one-thread-per-leaf kernel it replaces issued 8 800
// instructions one after the other.  17 296 leaves, k = 3: 57 -> 22 us (rocprofv3 means).
template <int K, int FX, class Buf>
__global__ __launch_bounds__(320, K <= 2 ? 3 : 2) void k_rhs_split_tree(const double *__restrict__ w,
                                                                       double *__restrict__ out,
                                                                       const double *__restrict__ dtp, TreeGrid g,
                                                                       long first, int mode, Mix mx,
                                                                       int *__restrict__ flag) {
  constexpr int N = (K + 1) * (K + 2) / 2, n1 = K + 1;
  constexpr Line<K> L{};
  __shared__ double sv[4 * N * 64];       // volume term [v][l][lane]
  __shared__ double sm[4 * 4 * n1 * 64];  // face moments [side][v][e][lane]
  __shared__ double st[3 * n1 * n1];      // P~_e at the nodes of a whole face, its low half, its high half
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = gridDim.x, xcd = blockIdx.x % 8, jb = blockIdx.x / 8;
  const long blk = (long)xcd * (nb / 8) + min(xcd, nb % 8) + jb;
  const long nl = g.nleaf;
  const bool own = first + 64 * blk + lane < nl;
  const unsigned leaf = (unsigned)min(first + 64 * blk + lane, nl - 1);
  using Cell = typename Buf::Cell;
  using Off = typename Buf::Off;
  const Cell cell = (Cell)8 * leaf;
  const Buf ws(w, nl, 4 * N), os(out, nl, 4 * N);
  if (threadIdx.x < 3 * n1 * n1) {
    const Line<K> &T = line_const<K>();
    const int h = threadIdx.x / (n1 * n1), r = threadIdx.x % (n1 * n1);
    st[threadIdx.x] = h == 0 ? T.p[r / n1][r % n1] : T.ph[h - 1][r / n1][r % n1];
  }
  __syncthreads();
  if (role == 0) {
    double wc[4][N];
    load_cell<4, N>(ws, cell, wc);
    if constexpr (K >= 3)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int l = 0; l < N; ++l) sv[(v * N + l) * 64 + lane] = wc[v][l];
    area_term<K, false>(
        [&](int v, int l) __attribute__((always_inline)) {
          if constexpr (K >= 3) return sv[(v * N + l) * 64 + lane];
          else return wc[v][l];
        },
        g.gamma - 1.0, [](int, int) __attribute__((always_inline)) { return 0.0; },
        [&](int v, const double(&r)[N]) __attribute__((always_inline)) {
#pragma unroll
          for (int l = 1; l < N; ++l) sv[(v * N + l) * 64 + lane] = r[l];
        });
  } else {
    const int side = role - 1;
    const int inf = g.info[(long)side * nl + leaf];
    const int kind = inf & 3, sub = (inf >> 2) & 1;
    // both table entries are read whatever the kind (-1 where there is no
    // neighbour): loads in a branch here had the compiler spill a register of
    // all lanes inside it (K = 3, 64-bit form: wrong fluxes)
    const int n0 = g.nb[(long)(2 * side) * nl + leaf], nh = g.nb[(long)(2 * side + 1) * nl + leaf];
    const unsigned j0 = kind == 1 ? leaf : (unsigned)n0, j1 = kind == 2 ? (unsigned)nh : leaf;
    double co[4][n1], m[4][n1];
    auto face = [&](auto A_, auto S_) __attribute__((always_inline)) {
      constexpr int A = decltype(A_)::value, S = decltype(S_)::value;
      double cn[4][n1];
      auto traces = [&](auto T_, Cell at, double (&c)[4][n1]) __attribute__((always_inline)) {
        constexpr int T = decltype(T_)::value;
#pragma unroll
        for (int v0 = 0; v0 < 4; v0 += 2) {
          double a[2][N];
          load_cell<2, N>(ws, at, a, (Off)(v0 * N) * ws.plane);
#pragma unroll
          for (int i = 0; i < 2; ++i) edge_coefs<K, A, T>(a[i], c[v0 + i]);
        }
      };
      traces(S_, cell, co);
      traces(std::integral_constant<int, 1 - S>{}, (Cell)8 * j0, cn);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < n1; ++e) m[v][e] = 0.0;
#pragma unroll 1
      for (int sb = 0; sb < 2; ++sb) {
        if (sb == 1) {
          if (!__any(kind == 2)) break;
          traces(std::integral_constant<int, 1 - S>{}, (Cell)8 * j1, cn);
        }
        const double *to = st + (kind == 2 ? (1 + sb) * n1 * n1 : 0), *tn = st + (kind == 3 ? (1 + sub) * n1 * n1 : 0);
        const double half = kind == 2 ? 0.5 : (sb == 0 ? 1.0 : 0.0);
#pragma unroll
        for (int i = 0; i < n1; ++i) {
          double UO[4], UN[4], f[4], p[n1];
#pragma unroll
          for (int e = 0; e < n1; ++e) p[e] = to[i * n1 + e];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double u = co[v][0];
#pragma unroll
            for (int e = 1; e < n1; ++e) u = fma(co[v][e], p[e], u);
            UO[v] = u;
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double u = cn[v][0];
#pragma unroll
            for (int e = 1; e < n1; ++e) u = fma(cn[v][e], tn[i * n1 + e], u);
            UN[v] = kind == 1 ? UO[v] : u;
          }
          if constexpr (S == 1) hllc_line<2, A, FX>(UO, UN, g.gamma, f);
          else hllc_line<2, A, FX>(UN, UO, g.gamma, f);
          const double wr = half * L.w[i];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double fv = sb == 0 || kind == 2 ? f[v] * wr : 0.0;
            m[v][0] += fv;
#pragma unroll
            for (int e = 1; e < n1; ++e) m[v][e] = fma(fv, p[e], m[v][e]);
          }
          DG_FENCE;
        }
      }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if (side == 0) face(I0{}, I0{});
    else if (side == 1) face(I0{}, I1{});
    else if (side == 2) face(I1{}, I0{});
    else face(I1{}, I1{});
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int e = 0; e < n1; ++e) sm[((side * 4 + v) * n1 + e) * 64 + lane] = m[v][e];
  }
  double wo[N], y0[N];
  const Buf ys(mode != 0 && mx.n > 0 ? mx.y[0] : w, nl, 4 * N);
  const int var = role < 4 ? role : 3;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    wo[l] = ws.load(cell, (Off)(var * N + l) * ws.plane);
    y0[l] = ys.load(cell, (Off)(var * N + l) * ws.plane);
  }
  __syncthreads();
  if (role == 4) return;

  double acc[N];
  acc[0] = 0.0;
#pragma unroll
  for (int l = 1; l < N; ++l) acc[l] = sv[(role * N + l) * 64 + lane];
  auto lift = [&](auto A_, auto S_) __attribute__((always_inline)) {
    constexpr int A = decltype(A_)::value, S = decltype(S_)::value;
    double mm[n1];
#pragma unroll
    for (int e = 0; e < n1; ++e) mm[e] = sm[(((2 * A + S) * 4 + role) * n1 + e) * 64 + lane];
    edge_lift<K, A, S>(mm, acc);
  };
  lift(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
  lift(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
  lift(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});
  lift(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
  if (!own) return;
  const double fac = g.fac0 * (double)(1 << g.lev[leaf]);
  const double cldt = mode == 0 ? 0.0 : mx.cl * *dtp;
  bool bad = false;
  Off off = (Off)(role * N) * os.plane;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    const double Lv = fac * acc[l];
    bad |= Lv != Lv;
    double o = Lv;
    if (mode != 0) {
      o = fma(cldt, Lv, mx.cu * wo[l]);
      if (mx.n > 0) o = fma(mx.a[0], y0[l], o);
      if (mx.n > 1) o = mix_tail(mx, o, (long)(role * N + l) * nl + leaf, 1);
    }
    os.store(o, cell, off);
    off += os.plane;
  }
  if (bad) atomicOr(flag, FLAG_NAN);
}

}  // namespace dg

// FP64 on 2D grids without a refined box or a tree, unless the configuration
// asks for a tile shape of the other kernel (tile2d) or has gravity at k = 4;
// states below 4 GB (32-bit byte offsets).  Faster at every size measured,
// 32^2 to 512^2.
bool dg::split2d_takes(const dg_ctx *c) {
  if (c->sh.d != 2 || c->amr || c->tree || c->cfg.precision != DG_FP64 || c->tile_small >= 0) return false;
  if (c->gravity && c->sh.k > 3) return false;
  return c->ncell * 8 * c->sh.nv * c->sh.N < (1LL << 32);
}

int dg::launch_split2d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                       const RateOp &ro, hipStream_t s) {
  SplitGrid g;
  g.nx = (int)c->nx;
  g.ny = (int)c->ny;
  g.nc = c->ncell;
  bool per = true;
  for (int a = 0; a < 2; ++a) {
    g.wall[a] = c->cfg.bc[a] == DG_BC_TRANSMISSIVE;
    per = per && !g.wall[a];
  }
  g.fac = 2.0 / c->dx / 4.0;
  g.gamma = c->cfg.gamma;
  g.columns = (long)(g.nx + 1) * g.ny;
  RateOp r = ro;
  if (r.op == RATE_FOLD && c->gravity) {
    r.gmax = c->gmax;
    r.gk = c->grav_k;
  }
  const dim3 nb((unsigned)((g.columns + 62) / 63));
  auto go = [&](auto K_, auto FX_) {
    constexpr int K = decltype(K_)::value, FX = decltype(FX_)::value;
    if (c->gravity) {
      if constexpr (K <= 3)
        hipLaunchKernelGGL((k_rhs_split2d<K, FX, false, true>), nb, dim3(256), 0, s, w, out, dt, g, mode, mx, c->flag, r, c->grav);
    } else if (per) {
      hipLaunchKernelGGL((k_rhs_split2d<K, FX, true, false>), nb, dim3(256), 0, s, w, out, dt, g, mode, mx, c->flag, r, nullptr);
    } else {
      hipLaunchKernelGGL((k_rhs_split2d<K, FX, false, false>), nb, dim3(256), 0, s, w, out, dt, g, mode, mx, c->flag, r, nullptr);
    }
  };
  auto pick = [&](auto K_) {
    if (c->cfg.flux == DG_HLLC_DAVIS) go(K_, std::integral_constant<int, DG_HLLC_DAVIS>{});
    else go(K_, std::integral_constant<int, DG_HLLC_BATTEN>{});
  };
  switch (c->sh.k) {
    case 1: pick(std::integral_constant<int, 1>{}); break;
    case 2: pick(std::integral_constant<int, 2>{}); break;
    case 3: pick(std::integral_constant<int, 3>{}); break;
    default: pick(std::integral_constant<int, 4>{}); break;
  }
  return (int)hipGetLastError();
}

int dg::launch_split_tree(const dg_ctx *c, const TreeGrid &g, const double *w, double *out, const double *dt, int mode,
                          const Mix &mx, hipStream_t s) {
  auto go = [&](auto K_) {
    constexpr int K = decltype(K_)::value;
    // byte offsets of 32 bits in the state (below 4 GB), else in each plane
    // (below 2^29 leaves), else of 64 bits (at k = 3 a state and its stage would
    // not fit the card)
    auto pick = [&](auto B_) {
      using Buf = std::remove_pointer_t<decltype(B_)>;
      return c->cfg.flux == DG_HLLC_DAVIS ? k_rhs_split_tree<K, DG_HLLC_DAVIS, Buf> : k_rhs_split_tree<K, DG_HLLC_BATTEN, Buf>;
    };
    auto kernel = pick((StateBuf *)nullptr);
    if ((long long)g.nleaf * 8 * c->sh.nv * c->sh.N >= (1LL << 32)) kernel = pick((StatePlanes *)nullptr);
    if (g.nleaf >= (1L << 29)) {
      if constexpr (K == 3) return (int)hipErrorOutOfMemory;
      else kernel = pick((StatePtr *)nullptr);
    }
    constexpr long most = launch_items(320);
    for (long first = 0; first < g.nleaf; first += most)
      hipLaunchKernelGGL(kernel, dim3((unsigned)((std::min(most, g.nleaf - first) + 63) / 64)), dim3(320), 0, s, w, out, dt,
                         g, first, mode, mx, c->flag);
    return (int)hipGetLastError();
  };
  if (c->sh.k == 1) return go(std::integral_constant<int, 1>{});
  if (c->sh.k == 2) return go(std::integral_constant<int, 2>{});
  return go(std::integral_constant<int, 3>{});
}
