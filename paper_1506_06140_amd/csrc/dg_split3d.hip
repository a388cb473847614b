// 3D right-hand side + stage, the work of 63 cells split over four waves
// (FP64; uniform grids and the refined box).
#include "dg_march.h"
#include "dg_rules.h"

namespace dg {

// One Cartesian block of cells: the grid, or the coarse or the fine block of
// a refined box.
struct Split3Part {
  int n[3];
  int wall[3];
  double fac;        // (2/dx) 2^-d
  long nc;
  long base;         // its state within the whole state, in doubles
  long columns;      // (nx + 1) ny
  long planes;       // blocks of 63 columns, times nz
};
struct Split3Grid {
  Split3Part p[2];
  int lo[3], hi[3];  // base cells under the fine block
  long total;        // planes of both parts
  long doubles;      // the whole state
  double gamma;
};

// A cell beside a face: where its state is, and what it is.
struct CellRef {
  unsigned off, stride;  // bytes: its first weight, one (variable, mode) plane
  int i[3];
  bool ghost;            // beyond a wall: the other side's trace
  bool hole;             // a coarse cell under the fine block
  bool coarse;           // a coarse cell beside a fine one
};

// x is formed here (not moved behind a branch, which would keep its operands
// alive)
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// c (2D, degree <= K, order of mode_index<2>) restricted to one quarter of
// the face: c'[j] = sum_e R[e][j] c[e] along each axis, s1, s2 = +-1 the half
// along the first and second axis.
template <int K>
__device__ __forceinline__ void restrict_face(double (&c)[(K + 1) * (K + 2) / 2], double s1, double s2) {
#pragma clang fp contract(off)
  constexpr Line<K> L{};
  static_for<0, K + 1>([&](auto J_) {
    constexpr int j = decltype(J_)::value;
    static_for<0, K + 1 - j>([&](auto F_) {
      constexpr int f = decltype(F_)::value;
      double ev = c[mode_index<2>(j, f, 0)] * L.rh[j][j], od = 0.0;
      static_for<j + 1, K + 1 - f>([&](auto E_) {
        constexpr int e = decltype(E_)::value;
        if constexpr ((e + j) % 2) od = fma(c[mode_index<2>(e, f, 0)], L.rh[e][j], od);
        else ev = fma(c[mode_index<2>(e, f, 0)], L.rh[e][j], ev);
      });
      c[mode_index<2>(j, f, 0)] = fma(s1, od, ev);
    });
  });
  static_for<0, K + 1>([&](auto J_) {
    constexpr int j = decltype(J_)::value;
    static_for<0, K + 1 - j>([&](auto F_) {
      constexpr int f = decltype(F_)::value;
      double ev = c[mode_index<2>(f, j, 0)] * L.rh[j][j], od = 0.0;
      static_for<j + 1, K + 1 - f>([&](auto E_) {
        constexpr int e = decltype(E_)::value;
        if constexpr ((e + j) % 2) od = fma(c[mode_index<2>(f, e, 0)], L.rh[e][j], od);
        else ev = fma(c[mode_index<2>(f, e, 0)], L.rh[e][j], ev);
      });
      c[mode_index<2>(f, j, 0)] = fma(s2, od, ev);
    });
  });
}
// face_coefs with the axis and the side (s = -1, +1) as uniform run-time values
template <int K>
__device__ __forceinline__ void side_trace(const double (&w)[(K + 1) * (K + 2) * (K + 3) / 6], int axis, double s,
                                           double (&c)[(K + 1) * (K + 2) / 2]) {
#pragma clang fp contract(off)
  constexpr Line<K> L{};
  auto go = [&](auto A_) __attribute__((always_inline)) {
    constexpr int A = decltype(A_)::value;
    static_for<0, (K + 1) * (K + 2) / 2>([&](auto J_) {
      constexpr int j = decltype(J_)::value, e1 = mode_exp<2>(j, 0), e2 = mode_exp<2>(j, 1);
      double t = 0.0, o = 0.0;
      static_for<0, K + 1>([&](auto N_) {
        constexpr int n = decltype(N_)::value;
        if constexpr (n + e1 + e2 <= K) {
          constexpr int l = A == 0 ? mode_index<3>(n, e1, e2) : A == 1 ? mode_index<3>(e1, n, e2) : mode_index<3>(e1, e2, n);
          if constexpr (n == 0) t = w[l];
          else if constexpr (n == 1) o = w[l] * L.b[1];
          else if constexpr (n == 2) t = fma(w[l], L.b[2], t);
          else o = fma(w[l], L.b[3], o);
        }
      });
      c[j] = fma(s, o, t);
      pin(c[j]);
    });
  };
  if (axis == 0) go(std::integral_constant<int, 0>{});
  else if (axis == 1) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 2>{});
}
// acc -+= the face's outward flux moments, side s = -1 (low) or +1 (uniform)
template <int K, int A>
__device__ __forceinline__ void side_lift(const double (&m)[(K + 1) * (K + 2) / 2], double s,
                                          double (&acc)[(K + 1) * (K + 2) * (K + 3) / 6]) {
  constexpr Line<K> L{};
  double me[(K + 1) * (K + 2) / 2];
#pragma unroll
  for (int j = 0; j < (K + 1) * (K + 2) / 2; ++j) me[j] = -s * m[j];
  static_for<0, (K + 1) * (K + 2) * (K + 3) / 6>([&](auto L_) {
    constexpr int l = decltype(L_)::value, ex = mode_exp<3>(l, 0), ey = mode_exp<3>(l, 1), ez = mode_exp<3>(l, 2);
    constexpr int n = A == 0 ? ex : A == 1 ? ey : ez, e1 = A == 0 ? ey : ex, e2 = A == 2 ? ey : ez;
    constexpr int j = mode_index<2>(e1, e2, 0);
    acc[l] = n % 2 ? fma(m[j], -L.b[n], acc[l]) : fma(me[j], L.b[n], acc[l]);
  });
}
// exchanges variables 1 and 1 + axis (uniform): the solver's normal momentum
// is variable 1 whatever the axis, so its code is there once
template <int N2>
__device__ __forceinline__ void swap_normal(double (&c)[5][N2], int axis) {
  auto go = [&](auto A_) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < N2; ++j) {
      const double x = c[1][j];
      c[1][j] = c[1 + decltype(A_)::value][j];
      c[1 + decltype(A_)::value][j] = x;
      pin(c[1][j]);
      pin(c[1 + decltype(A_)::value][j]);
    }
  };
  if (axis == 1) go(std::integral_constant<int, 1>{});
  else if (axis == 2) go(std::integral_constant<int, 2>{});
}
// moments against the whole face's polynomials from those against a
// quarter's, with the quarter's share 1/4 of the area: the transpose
template <int K>
__device__ __forceinline__ void restrict_face_t(double (&m)[(K + 1) * (K + 2) / 2], double s1, double s2) {
  constexpr Line<K> L{};
  static_for<0, K + 1>([&](auto I_) {
    constexpr int e = K - decltype(I_)::value;
    static_for<0, K + 1 - e>([&](auto F_) {
      constexpr int f = decltype(F_)::value;
      double ev = m[mode_index<2>(f, e, 0)] * L.rh[e][e], od = 0.0;
      static_for<0, e>([&](auto J_) {
        constexpr int j = decltype(J_)::value;
        if constexpr ((e + j) % 2) od = fma(m[mode_index<2>(f, j, 0)], L.rh[e][j], od);
        else ev = fma(m[mode_index<2>(f, j, 0)], L.rh[e][j], ev);
      });
      m[mode_index<2>(f, e, 0)] = fma(s2, od, ev);
    });
  });
  static_for<0, K + 1>([&](auto I_) {
    constexpr int e = K - decltype(I_)::value;
    static_for<0, K + 1 - e>([&](auto F_) {
      constexpr int f = decltype(F_)::value;
      double ev = m[mode_index<2>(e, f, 0)] * L.rh[e][e], od = 0.0;
      static_for<0, e>([&](auto J_) {
        constexpr int j = decltype(J_)::value;
        if constexpr ((e + j) % 2) od = fma(m[mode_index<2>(j, f, 0)], L.rh[e][j], od);
        else ev = fma(m[mode_index<2>(j, f, 0)], L.rh[e][j], ev);
      });
      m[mode_index<2>(e, f, 0)] = 0.25 * fma(s1, od, ev);
    });
  });
}

// One plane of the volume integral: from the state's 2D coefficients at
// z = z_i the moments M[t] of the nine distinct fluxes (xx xy xz yy yz zz, hx
// hy hz) against the plane's polynomials of degree <= K - 1.
template <int K>
__device__ __forceinline__ void plane_moments(const double (&c)[5][(K + 1) * (K + 2) / 2], double gm1,
                                              double (&M)[9][K * (K + 1) / 2]) {
  constexpr int n1 = K + 1, NP = K * (K + 1) / 2;
  const Line<K> &T = line_const<K>();
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < NP; ++j) M[t][j] = 0.0;
#pragma unroll 1
  for (int iy = 0; iy < n1; ++iy) {
    double py[n1];
#pragma unroll
    for (int e = 0; e < n1; ++e) py[e] = T.p[iy][e];
    const double wy = T.w[iy];
    double U[5][n1];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double c1[n1];
      static_for<0, n1>([&](auto E_) {
        constexpr int ex = decltype(E_)::value;
        double t = c[v][mode_index<2>(ex, 0, 0)];
        static_for<1, n1 - ex>([&](auto G_) {
          constexpr int ey = decltype(G_)::value;
          t = fma(c[v][mode_index<2>(ex, ey, 0)], py[ey], t);
        });
        c1[ex] = t;
      });
      line_values<K, K>(c1, U[v]);
    }
    DG_FENCE;
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
      static_for<0, NP>([&](auto J_) {
        constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
        M[t][j] = fma(s[ex], wy * py[ey], M[t][j]);
      });
    }
    DG_FENCE;
  }
}

// acc += variable v's volume term of one plane: pz[e] = w_i P~_e(z_i), dz[e] =
// w_i P~_e'(z_i).  The mass flux is the momentum, a polynomial of the cell:
// its moments over the plane are 2^2 times the momentum's coefficients.
template <int K, int V>
__device__ __forceinline__ void plane_lift(const double (&M)[9][K * (K + 1) / 2],
                                           const double (&c)[5][(K + 1) * (K + 2) / 2], const double (&pz)[K + 1],
                                           const double (&dz)[K + 1], double (&acc)[(K + 1) * (K + 2) * (K + 3) / 6]) {
  constexpr Line<K> L{};
  constexpr int N2 = (K + 1) * (K + 2) / 2, N = (K + 1) * (K + 2) * (K + 3) / 6;
  auto mom = [&](auto A_, auto J_) __attribute__((always_inline)) {
    constexpr int a = decltype(A_)::value, j = decltype(J_)::value;
    constexpr int t = V == 1   ? a
                      : V == 2 ? (a == 0 ? 1 : a == 1 ? 3 : 4)
                      : V == 3 ? (a == 0 ? 2 : a == 1 ? 4 : 5)
                               : 6 + a;
    if constexpr (V == 0) return 4.0 * c[1 + a][j];
    else return M[t][j];
  };
  double q[N2];
  static_for<0, N2>([&](auto J_) {
    constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
    double t = 0.0;
    static_for<0, ex>([&](auto E_) {
      constexpr int e = decltype(E_)::value;
      if constexpr ((ex - e) % 2) {
        constexpr double dc = L.dc[ex][e];
        t = fma(mom(std::integral_constant<int, 0>{}, std::integral_constant<int, mode_index<2>(e, ey, 0)>{}), dc, t);
      }
    });
    static_for<0, ey>([&](auto E_) {
      constexpr int e = decltype(E_)::value;
      if constexpr ((ey - e) % 2) {
        constexpr double dc = L.dc[ey][e];
        t = fma(mom(std::integral_constant<int, 1>{}, std::integral_constant<int, mode_index<2>(ex, e, 0)>{}), dc, t);
      }
    });
    q[j] = t;
  });
  static_for<1, N>([&](auto L_) {
    constexpr int l = decltype(L_)::value, ex = mode_exp<3>(l, 0), ey = mode_exp<3>(l, 1), ez = mode_exp<3>(l, 2);
    double t = acc[l];
    if constexpr (ex + ey > 0) t = fma(q[mode_index<2>(ex, ey, 0)], pz[ez], t);
    if constexpr (ez > 0)
      t = fma(mom(std::integral_constant<int, 2>{}, std::integral_constant<int, mode_index<2>(ex, ey, 0)>{}), dz[ez], t);
    acc[l] = t;
  });
}

// f(std::integral_constant<int, I>) for the runtime (uniform) i in [0, E)
template <int E, int I = 0, class F>
__device__ __forceinline__ void pick(int i, F &&f) {
  if constexpr (I < E) {
    if (i == I) f(std::integral_constant<int, I>{});
    else pick<E, I + 1>(i, f);
  }
}

// 3D right-hand side and stage of uniform grids (k = 3) and of the refined box.
//
// A workgroup is one compute unit's four waves; lane by lane they share 64
// positions of rows of nx + 1 (63 owned cells: x face px lies between cells
// px - 1 and px, each solved once, its moments handed to the lane below), and
// march along z.  Each wave takes one face of its lane's cell - x low, y low,
// y high, z high - and one of the four planes z = z_i of the cell's volume
// quadrature, so all four do the same amount of work: at k = 3 about 3100
// FP64 operations for a face's 16 Riemann solves and 1400 for a plane's 16
// points, everything contracted one axis at a time.  The upper z face's
// moments start the next plane's accumulators.  A cell's 100 accumulators sit
// in LDS (50 KB), as do each wave's own traces (4 x 25 KB); wave i adds to
// variable i, i + 1, ... in five steps with a barrier between, so the order of
// the additions is fixed.  512 registers a lane (one wave per SIMD): the
// neighbour's 100 weights are in flight while the plane is computed.
// The solver is there once, with the normal momentum as variable 1 for every
// axis: with three copies of it and the box's faces in the same kernel the
// code outgrew the 64 KB instruction cache that two compute units share
// (64^3 box at k = 3: 2310 us a stage, 1150 misses per cache).
// Planes go to the workgroups, one per compute unit (150 KB of LDS), in equal
// contiguous runs; a run or a column that starts without a plane below it
// solves that z face first (pass 0).
// Box: the coarse and the fine block are two such grids in one launch.  A fine
// cell's coarse neighbour's trace is restricted to its quarter of the face; a
// coarse cell's faces with the fine block get a zero flux here and theirs from
// k_box_faces.  Both form the traces and the flux with the same code, so both
// sides of a face see the same flux.
// Bound by issue at one wave per SIMD: vector ALU busy 40 % of the cycles, 24 %
// of them on loads and barriers, 20 % on dependent results.  One launch, FP64
// MFMA kernel -> this: k = 3, 8^3 67 -> 54 us, 32^3 142 -> 141, 64^3 1107 -> 629,
// 128^3 8581 -> 5149; a box of twice as many cells as its base grid, k = 3,
// 64^3 2469 -> 1440 (both kernels), 24^3 163 -> 146, k = 2, 96 x 96 x 64 2178 ->
// 1517, 32^3 145 -> 138, 8^3 58 -> 44.
template <int K, int FX, bool AMR>
__global__ __launch_bounds__(256, 1) void k_rhs_split3d(const double *__restrict__ w, double *__restrict__ out,
                                                        const double *__restrict__ dtp, Split3Grid g, int mode, Mix mx,
                                                        int *__restrict__ flag) {
  constexpr int N = (K + 1) * (K + 2) * (K + 3) / 6, N2 = (K + 1) * (K + 2) / 2, n1 = K + 1;
  constexpr int NP = K * (K + 1) / 2, NO = (5 * N + 3) / 4;
  __shared__ double sa[5 * N * 64];       // V - S of the 64 cells: [v][l][lane]
  __shared__ double sx[4 * 5 * N2 * 64];  // per wave: its face's low traces, [v][j][lane]
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // XCD b mod 8 takes a contiguous band of the planes
  const int G = gridDim.x, xcd = blockIdx.x % 8, jb = blockIdx.x / 8;
  const long b = (long)xcd * (G / 8) + min(xcd, G % 8) + jb;
  const long p0 = g.total * b / G, p1 = g.total * (b + 1) / G;
  const Line<K> &T = line_const<K>();
  const double gm1 = g.gamma - 1.0;
  const StateBuf ws(w, g.doubles, 1), os(out, g.doubles, 1);
  const StateBuf ys(mode != 0 && mx.n > 0 ? mx.y[0] : w, g.doubles, 1);
  const double cldt = mode == 0 ? 0.0 : mx.cl * *dtp, cu = mode == 0 ? 0.0 : mx.cu;
  const int ny0 = mode == 0 ? 0 : mx.n;
  bool bad = false;
  double *const sxw = sx + role * (5 * N2 * 64);
  auto low = [&](int v, int j) __attribute__((always_inline)) -> double & { return sxw[(v * N2 + j) * 64 + lane]; };
  auto acc_row = [&](int v, double (&r)[N]) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < N; ++l) r[l] = sa[(v * N + l) * 64 + lane];
  };
  auto set_acc = [&](int v, const double (&r)[N]) __attribute__((always_inline)) {
#pragma unroll
    for (int l = 0; l < N; ++l) sa[(v * N + l) * 64 + lane] = r[l];
  };
  const int iz = min(role, K);  // this wave's plane of the volume integral
  double pz[n1], wpz[n1], wdz[n1];
#pragma unroll
  for (int e = 0; e < n1; ++e) {
    pz[e] = T.p[iz][e];
    wpz[e] = T.w[iz] * pz[e];
    double d = 0.0;
#pragma unroll
    for (int j = 0; j < e; ++j) d = fma(T.dc[e][j], pz[j], d);
    wdz[e] = T.w[iz] * d;
  }

  auto in_hole = [&](int x, int y, int zz) {
    return x >= g.lo[0] && x < g.hi[0] && y >= g.lo[1] && y < g.hi[1] && zz >= g.lo[2] && zz < g.hi[2];
  };
  // the cell at (x, y, zz) of part P, at most one index one past its range: a
  // periodic or wall neighbour, or (fine block) the coarse cell beside it
  // (the box keeps a cell's distance from the domain's faces)
  auto ref = [&](const Split3Part &P, bool fine, int x, int y, int zz) __attribute__((always_inline)) {
    CellRef r;
    r.i[0] = x;
    r.i[1] = y;
    r.i[2] = zz;
    r.ghost = r.hole = r.coarse = false;
    bool beyond = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const bool lo = r.i[a] < 0, hi = r.i[a] >= P.n[a];
      beyond |= lo | hi;
      if (!fine) {
        const bool wall = P.wall[a];
        r.ghost |= wall && (lo || hi);
        r.i[a] = lo ? (wall ? 0 : P.n[a] - 1) : hi ? (wall ? P.n[a] - 1 : 0) : r.i[a];
      }
    }
    unsigned nx = (unsigned)P.n[0], ny = (unsigned)P.n[1], base = (unsigned)P.base;
    r.stride = 8u * (unsigned)P.nc;
    if (AMR && fine) {
      r.coarse = beyond;
      if (beyond) {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.i[a] = g.lo[a] + (r.i[a] >> 1);
        nx = (unsigned)g.p[0].n[0];
        ny = (unsigned)g.p[0].n[1];
        base = 0;
        r.stride = 8u * (unsigned)g.p[0].nc;
      }
    } else if (AMR) {
      r.hole = in_hole(r.i[0], r.i[1], r.i[2]);
    }
    r.off = 8u * (base + ((unsigned)r.i[2] * ny + (unsigned)r.i[1]) * nx + (unsigned)r.i[0]);
    return r;
  };

#pragma unroll 1
  for (long p = p0; p < p1; ++p) {
    const bool fine = AMR && p >= g.p[0].planes;
    const Split3Part &P = g.p[fine ? 1 : 0];
    const long q = fine ? p - g.p[0].planes : p;
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int cb = (int)(q / nz), z = (int)(q % nz);
    const long e0 = 63L * cb + lane;
    const unsigned e = (unsigned)min(e0, P.columns - 1);
    const int px = (int)(e % (unsigned)(nx + 1)), iy = (int)(e / (unsigned)(nx + 1)), cx = min(px, nx - 1);
    const bool own = px < nx && lane < 63 && e0 < P.columns;
    const unsigned stride = 8u * (unsigned)P.nc;
    const bool fresh = p == p0 || z == 0;
#pragma unroll 1
    for (int ps = fresh ? 0 : 1; ps < 2; ++ps) {
      // pass 0: the low z face of a column's first plane (all four waves, wave
      // 3 keeps it); pass 1: the plane
      const bool last = ps == 1;
      const int type = last ? role : 4;  // x low, y low, y high, z high; z low
      const CellRef A = ref(P, fine, type == 0 ? px - 1 : cx, iy - (type == 1), z - (type == 4));
      const CellRef B = ref(P, fine, type == 0 ? px : cx, iy + (type == 2), z + (type == 3));
      const int axis = type == 0 ? 0 : type < 3 ? 1 : 2;
      const bool drop = AMR && (A.hole || B.hole);
      const double s1 = ((axis == 0 ? iy : cx) & 1) ? 1.0 : -1.0, s2 = ((axis == 2 ? iy : z) & 1) ? 1.0 : -1.0;
      // all of a cell's weights in flight at once
      auto fetch = [&](double (&c)[5][N], unsigned o, unsigned str) __attribute__((always_inline)) {
        unsigned so = 0, st = stride;
        asm volatile("" : "+s"(st));  // its multiples are formed here, not kept through the loop
#pragma unroll
        for (int v = 0; v < 5; ++v)
#pragma unroll
          for (int l = 0; l < N; ++l) {
            c[v][l] = ws.load(o, so);
            if constexpr (AMR) o += str;
            else so += st;
          }
        DG_FENCE;
      };
      // the traces in LDS restricted in the lanes with on: a coarse cell beside fine ones
      auto quarter = [&](bool on) __attribute__((always_inline)) {
        if (!__any(on)) return;
#pragma unroll 1
        for (int v = 0; v < 5; ++v) {
          double t[N2], x[N2];
#pragma unroll
          for (int j = 0; j < N2; ++j) x[j] = t[j] = low(v, j);
          restrict_face<K>(x, s1, s2);
#pragma unroll
          for (int j = 0; j < N2; ++j) low(v, j) = on ? x[j] : t[j];
        }
      };
      const bool upper = type < 2 || type == 4;  // the own cell is the face's upper one
      // the own cell: its plane z_iz of the volume integral, its trace to LDS
      double c2[5][N2];
      {
        double wc[5][N];
        fetch(wc, upper ? B.off : A.off, upper ? B.stride : A.stride);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double(&c)[N] = wc[v];
          double t[N2];
          static_for<0, N2>([&](auto J_) {
            constexpr int j = decltype(J_)::value, ex = mode_exp<2>(j, 0), ey = mode_exp<2>(j, 1);
            double x = c[mode_index<3>(ex, ey, 0)];
            static_for<1, n1 - ex - ey>([&](auto G_) {
              constexpr int ez = decltype(G_)::value;
              x = fma(c[mode_index<3>(ex, ey, ez)], pz[ez], x);
            });
            c2[v][j] = x;
            pin(c2[v][j]);
          });
          side_trace<K>(c, axis, upper ? -1.0 : 1.0, t);
          const int vp = v == 1 ? 1 + axis : v == 1 + axis ? 1 : v;
#pragma unroll
          for (int j = 0; j < N2; ++j) low(vp, j) = t[j];
          DG_FENCE;
        }
        if (AMR) quarter(upper ? B.coarse : A.coarse);
      }
      double nb[5][N], M[9][NP];
      if (last && (n1 == 4 || role < n1)) plane_moments<K>(c2, gm1, M);
      fetch(nb, upper ? A.off : B.off, upper ? A.stride : B.stride);
      if (last) {
        __syncthreads();
#pragma unroll 1
        for (int s = 0; s < 5; ++s) {
          const int vr = role + s < 5 ? role + s : role + s - 5;
          if (n1 == 4 || role < n1)
            pick<5>(vr, [&](auto V_) __attribute__((always_inline)) {
              constexpr int v = decltype(V_)::value;
              double r[N];
              acc_row(v, r);
              plane_lift<K, v>(M, c2, wpz, wdz, r);
              set_acc(v, r);
            });
          __syncthreads();
        }
        DG_FENCE;
      }
      double m[5][N2];
      {
        // the own traces move to registers, the neighbour's take their place
        double ch[5][N2];
        const bool og = upper ? A.ghost : B.ghost;  // no neighbour: a wall
        const bool pg = upper ? B.ghost : A.ghost;  // (x: the position past the row's end)
#pragma unroll
        for (int v = 0; v < 5; ++v)
#pragma unroll
          for (int j = 0; j < N2; ++j) ch[v][j] = low(v, j);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double(&c)[N] = nb[v];
          double t[N2];
          side_trace<K>(c, axis, upper ? 1.0 : -1.0, t);
          const int vp = v == 1 ? 1 + axis : v == 1 + axis ? 1 : v;
#pragma unroll
          for (int j = 0; j < N2; ++j) low(vp, j) = t[j];
          DG_FENCE;
        }
        if (AMR) quarter(upper ? A.coarse : B.coarse);
        if (__any(og || pg)) {
#pragma unroll
          for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int j = 0; j < N2; ++j) {
              const double o = ch[v][j], t = low(v, j);
              low(v, j) = og ? o : t;
              ch[v][j] = pg ? t : o;
              pin(ch[v][j]);
            }
        }
        if (!upper) {
#pragma unroll
          for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int j = 0; j < N2; ++j) {
              const double o = ch[v][j];
              ch[v][j] = low(v, j);
              low(v, j) = o;
              pin(ch[v][j]);
            }
        }
        DG_FENCE;
        face_flux<K, 0, FX>(low, ch, g.gamma, m);
        swap_normal(m, axis);
        if (AMR && __any(drop)) {
#pragma unroll
          for (int v = 0; v < 5; ++v)
#pragma unroll
            for (int j = 0; j < N2; ++j) m[v][j] = drop ? 0.0 : m[v][j];
        }
      }
      // the upper cell's accumulators start from the z face's flux
      auto start = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          double r[N];
#pragma unroll
          for (int l = 0; l < N; ++l) r[l] = 0.0;
          face_lift<K, 2, 0>(m[v], r);
          set_acc(v, r);
          DG_FENCE;
        }
      };
      if (ps == 0) {
        if (role == 3) start();
        continue;
      }
      const unsigned cell = 8u * ((unsigned)P.base + (unsigned)(z * ny + iy) * (unsigned)nx + (unsigned)cx);
#pragma unroll 1
      for (int s = 0; s < 5; ++s) {
        const int vr = role + s < 5 ? role + s : role + s - 5;
        pick<5>(vr, [&](auto V_) __attribute__((always_inline)) {
          constexpr int v = decltype(V_)::value;
          double r[N];
          acc_row(v, r);
          if (axis == 0) {
            double h[N2];
#pragma unroll
            for (int j = 0; j < N2; ++j) h[j] = lane_above(m[v][j]);
            face_lift<K, 0, 0>(m[v], r);
            face_lift<K, 0, 1>(h, r);
          } else if (axis == 1) {
            side_lift<K, 1>(m[v], upper ? -1.0 : 1.0, r);
          } else {
            face_lift<K, 2, 1>(m[v], r);
          }
          set_acc(v, r);
        });
        __syncthreads();
      }
      const bool hole = AMR && !fine && in_hole(cx, iy, z);
      unsigned st = stride;
      asm volatile("" : "+s"(st));
      // this wave's NO rows of the 5 N; past the last one the last again, not
      // stored (no read may lie outside the state: a row's offset is the buffer
      // instruction's scalar one, which may be larger than what follows a small
      // fine block)
      const int row0 = role * NO;
      const unsigned off0 = (unsigned)row0 * st;
      auto next = [&](unsigned off, int i) __attribute__((always_inline)) {
        return 5 * N % 4 == 0 || row0 + i + 1 < 5 * N ? off + st : off;
      };
      double u[NO], y0[NO];
      {
        unsigned off = off0;
#pragma unroll
        for (int i = 0; i < NO; ++i) {
          u[i] = ws.load(cell, off);
          y0[i] = ys.load<NT>(cell, off);
          off = next(off, i);
        }
      }
      const double cl = hole ? 0.0 : cldt, a0 = mx.a[0];
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const int c = row0 + i;
        const double L = hole ? 0.0 : P.fac * sa[(5 * N % 4 == 0 ? c : min(c, 5 * N - 1)) * 64 + lane];
        bad |= own && L != L;
        const double o = fma(cl, L, cu * u[i]), o1 = fma(a0, y0[i], o);  // mix_out
        u[i] = mode == 0 ? L : ny0 > 0 ? o1 : o;
      }
#pragma unroll 1
      for (int k = 1; k < ny0; ++k) {
        const StateBuf yk(mx.y[k], g.doubles, 1);
        unsigned off = off0;
#pragma unroll
        for (int i = 0; i < NO; ++i) {
          u[i] = fma(mx.a[k], yk.load<NT>(cell, off), u[i]);
          off = next(off, i);
        }
      }
      unsigned off = off0;
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        if (own && (5 * N % 4 == 0 || row0 + i < 5 * N)) os.store<NT>(u[i], cell, off);
        off = next(off, i);
      }
      __syncthreads();
      if (role == 3) start();
    }
  }
  if (bad) atomicOr(flag, FLAG_NAN);
}

// The coarse cells' faces with the fine block: four lanes a face, one per
// quarter, each the solve that the fine cell beside it makes (the coarse trace
// restricted, the same code), its moments back on the whole face, summed over
// the four lanes and lifted onto the stage's output, to which k_rhs_split3d
// gave these faces a zero flux.  A coarse cell has one such face (the box is
// convex and a cell away from the domain's faces), so the order of the
// additions is fixed.
template <int K, int FX>
__global__ __launch_bounds__(64, 1) void k_box_faces(const double *__restrict__ w, double *__restrict__ out,
                                                     const double *__restrict__ dtp, Split3Grid g, int mode, double cl,
                                                     int *__restrict__ flag) {
  constexpr int N = (K + 1) * (K + 2) * (K + 3) / 6, N2 = (K + 1) * (K + 2) / 2;
  __shared__ double sx[5 * N2 * 64];
  const int lane = threadIdx.x;
  int blk = blockIdx.x, side = 0, n1 = 0, n2 = 0;
  for (; side < 6; ++side) {
    const int ax = side >> 1, t1 = ax == 0 ? 1 : 0, t2 = ax == 2 ? 1 : 2;
    n1 = g.hi[t1] - g.lo[t1];
    n2 = g.hi[t2] - g.lo[t2];
    const int nb = (n1 * n2 + 15) / 16;
    if (blk < nb) break;
    blk -= nb;
  }
  const int axis = side >> 1, t1 = axis == 0 ? 1 : 0, t2 = axis == 2 ? 1 : 2;
  const bool above = side & 1;  // the coarse cell is above the box
  const int face = 16 * blk + (lane >> 2), f = min(face, n1 * n2 - 1), b1 = lane & 1, b2 = (lane >> 1) & 1;
  const bool real = face < n1 * n2 && (lane & 3) == 0;
  const int j1 = f % n1, j2 = f / n1;
  const Split3Part &C = g.p[0], &F = g.p[1];
  auto cell_of = [&](const Split3Part &P, int a, int x1, int x2) {
    const int x = axis == 0 ? a : x1, y = axis == 1 ? a : axis == 0 ? x1 : x2, z = axis == 2 ? a : x2;
    return 8u * ((unsigned)P.base + ((unsigned)z * (unsigned)P.n[1] + (unsigned)y) * (unsigned)P.n[0] + (unsigned)x);
  };
  const unsigned co = cell_of(C, above ? g.hi[axis] : g.lo[axis] - 1, g.lo[t1] + j1, g.lo[t2] + j2);
  const unsigned fo = cell_of(F, above ? F.n[axis] - 1 : 0, 2 * j1 + b1, 2 * j2 + b2);
  const unsigned cs = 8u * (unsigned)C.nc, fs = 8u * (unsigned)F.nc;
  const double s1 = b1 ? 1.0 : -1.0, s2 = b2 ? 1.0 : -1.0;
  const StateBuf ws(w, g.doubles, 1), os(out, g.doubles, 1);
  auto low = [&](int v, int j) __attribute__((always_inline)) -> double & { return sx[(v * N2 + j) * 64 + lane]; };
  double tc[5][N2], tf[5][N2];
  unsigned oc = 0, of = 0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double a[N], b[N];
#pragma unroll
    for (int l = 0; l < N; ++l) {
      a[l] = ws.load(co, oc);
      b[l] = ws.load(fo, of);
      oc += cs;
      of += fs;
    }
    side_trace<K>(a, axis, above ? -1.0 : 1.0, tc[v]);
    side_trace<K>(b, axis, above ? 1.0 : -1.0, tf[v]);
    restrict_face<K>(tc[v], s1, s2);
    DG_FENCE;
  }
  swap_normal(tc, axis);
  swap_normal(tf, axis);
#pragma unroll
  for (int v = 0; v < 5; ++v)
#pragma unroll
    for (int j = 0; j < N2; ++j) {
      const double c = tc[v][j], x = tf[v][j];
      low(v, j) = above ? x : c;
      tf[v][j] = above ? c : x;
      pin(tf[v][j]);
    }
  double m[5][N2];
  face_flux<K, 0, FX>(low, tf, g.gamma, m);
  swap_normal(m, axis);
  const double scale = C.fac * (mode == 0 ? 1.0 : cl * *dtp);
  bool bad = false;
  unsigned off = 0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    restrict_face_t<K>(m[v], s1, s2);
#pragma unroll
    for (int j = 0; j < N2; ++j) {
      double t = m[v][j];
      t += __shfl_xor(t, 1);
      t += __shfl_xor(t, 2);
      m[v][j] = t;
      bad |= real && t != t;
    }
    double r[N], o[N];
    unsigned of2 = off;
#pragma unroll
    for (int l = 0; l < N; ++l) {
      r[l] = 0.0;
      o[l] = os.load(co, of2);
      of2 += cs;
    }
    pick<3>(axis, [&](auto A_) __attribute__((always_inline)) {
      side_lift<K, decltype(A_)::value>(m[v], above ? -1.0 : 1.0, r);
    });
#pragma unroll
    for (int l = 0; l < N; ++l) {
      if (real) os.store(fma(scale, r[l], o[l]), co, off);
      off += cs;
    }
    DG_FENCE;
  }
  if (bad) atomicOr(flag, FLAG_NAN);
}

}  // namespace dg

// FP64 in 3D without gravity, states below 4 GB (32-bit byte offsets), of the
// sizes where it is faster: the refined box at k = 2, 3, and uniform grids at
// k = 3 (k = 2 has the march and MFMA kernels; here 16^3 takes 30.2 us against
// MFMA's 27.7, 25 x 25 x 26 57.8 against 37.0).
bool dg::split3d_takes(const dg_ctx *c) {
  if (c->sh.d != 3 || c->sh.k < 2 || c->gravity || c->tree) return false;
  if (c->cfg.precision != DG_FP64 || c->cfg.path3d != DG_PATH3D_AUTO) return false;
  const long cells = c->amr ? c->ncc + c->ncf : c->ncell;
  if (cells * 8 * c->sh.nv * c->sh.N >= (1LL << 32)) return false;
  const long n[3] = {c->nx, c->ny, c->nz};
  if (c->amr) return split3d_box_faster(c->sh.k, n, c->nf);
  return c->sh.k == 3 && split3d_faster(n[0], n[1], n[2]);
}

int dg::launch_split3d(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                       hipStream_t s) {
  Split3Grid g;
  const int n[3] = {(int)c->nx, (int)c->ny, (int)c->nz};
  g.total = 0;
  for (int i = 0; i < 2; ++i) {
    Split3Part &p = g.p[i];
    for (int a = 0; a < 3; ++a) {
      p.n[a] = i == 0 ? n[a] : c->amr ? (int)c->nf[a] : 1;
      p.wall[a] = i == 0 && c->cfg.bc[a] == DG_BC_TRANSMISSIVE;
      g.lo[a] = c->amr ? c->lo[a] : 0;
      g.hi[a] = c->amr ? c->hi[a] : 0;
    }
    p.fac = 2.0 / (i == 0 ? c->dx : 0.5 * c->dx) / 8.0;
    p.nc = i == 0 ? (long)n[0] * n[1] * n[2] : c->amr ? c->ncf : 0;
    p.base = i == 0 ? 0 : g.p[0].nc * c->sh.nv * c->sh.N;
    p.columns = (long)(p.n[0] + 1) * p.n[1];
    p.planes = i == 0 || c->amr ? split_planes(p.n[0], p.n[1], p.n[2]) : 0;
    g.total += p.planes;
  }
  g.doubles = (g.p[0].nc + g.p[1].nc) * c->sh.nv * c->sh.N;
  g.gamma = c->cfg.gamma;
  const dim3 nb((unsigned)std::min(kCusPerGpu, g.total));
  auto go = [&](auto K_, auto FX_) {
    constexpr int K = decltype(K_)::value, FX = decltype(FX_)::value;
    if (c->amr) {
      unsigned faces = 0;
      for (int a = 0; a < 3; ++a)
        faces += 2u * (unsigned)(((g.hi[(a + 1) % 3] - g.lo[(a + 1) % 3]) * (g.hi[(a + 2) % 3] - g.lo[(a + 2) % 3]) + 15) / 16);
      hipLaunchKernelGGL((k_rhs_split3d<K, FX, true>), nb, dim3(256), 0, s, w, out, dt, g, mode, mx, c->flag);
      hipLaunchKernelGGL((k_box_faces<K, FX>), dim3(faces), dim3(64), 0, s, w, out, dt, g, mode, mx.cl, c->flag);
    } else if constexpr (K == 3) {  // split3d_takes: k = 2 for the box only
      hipLaunchKernelGGL((k_rhs_split3d<K, FX, false>), nb, dim3(256), 0, s, w, out, dt, g, mode, mx, c->flag);
    }
  };
  using B = std::integral_constant<int, DG_HLLC_BATTEN>;
  using V = std::integral_constant<int, DG_HLLC_DAVIS>;
  const bool dav = c->cfg.flux == DG_HLLC_DAVIS;
  if (c->sh.k == 2) dav ? go(std::integral_constant<int, 2>{}, V{}) : go(std::integral_constant<int, 2>{}, B{});
  else dav ? go(std::integral_constant<int, 3>{}, V{}) : go(std::integral_constant<int, 3>{}, B{});
  return (int)hipGetLastError();
}
