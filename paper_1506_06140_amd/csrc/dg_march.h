// What the sum-factorised stage kernels (dg_split2d.hip, dg_march3d.hip,
// dg_split3d.hip, dg_adjoint2d.hip) share.
#pragma once

#include "dg_line.h"

// Keeps the scheduler from interleaving across it: each phase's temporaries
// die before the next phase's are formed.
#define DG_FENCE __builtin_amdgcn_sched_barrier(0)

namespace dg {

// A state as a buffer: byte offsets of 32 bits (the launcher checks that the
// state is below 4 GB), the (variable, mode) plane as the scalar offset, so a
// load takes one vector register of address and no scalar base of its own.
struct StateBuf {
  using Cell = unsigned;
  using Off = unsigned;
  __amdgpu_buffer_rsrc_t r;
  unsigned plane;  // bytes of one (variable, mode) plane
  __device__ __forceinline__ StateBuf(const double *p, long nc, int planes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, (int)(unsigned)(nc * 8 * planes), 0x00027000)),
        plane((unsigned)nc * 8u) {}
  template <int AUX = 0>
  __device__ __forceinline__ double load(unsigned cell8, unsigned off) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_amdgcn_raw_buffer_load_b64(r, cell8, off, AUX);
    return __hiloint2double((int)x.y, (int)x.x);
  }
  template <int AUX = 0>
  __device__ __forceinline__ void store(double v, unsigned cell8, unsigned off) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = {(unsigned)__double2loint(v), (unsigned)__double2hiint(v)};
    __builtin_amdgcn_raw_buffer_store_b64(x, r, cell8, off, AUX);
  }
};
// A state whose planes are below 4 GB each: every plane a buffer of its own
// (scalar arithmetic), the cell its 32-bit byte offset.
struct StatePlanes {
  using Cell = unsigned;
  using Off = size_t;
  double *p;
  Off plane;
  __device__ __forceinline__ StatePlanes(const double *q, long nc, int) : p(const_cast<double *>(q)), plane((Off)nc * 8) {}
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t at(Off off) const {
    return __builtin_amdgcn_make_buffer_rsrc((char *)p + off, 0, (int)(unsigned)plane, 0x00027000);
  }
  template <int AUX = 0>
  __device__ __forceinline__ double load(Cell cell8, Off off) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_amdgcn_raw_buffer_load_b64(at(off), cell8, 0, AUX);
    return __hiloint2double((int)x.y, (int)x.x);
  }
  template <int AUX = 0>
  __device__ __forceinline__ void store(double v, Cell cell8, Off off) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = {(unsigned)__double2loint(v), (unsigned)__double2hiint(v)};
    __builtin_amdgcn_raw_buffer_store_b64(x, at(off), cell8, 0, AUX);
  }
};
// A state of any size: 64-bit byte offsets in vector registers.
struct StatePtr {
  using Cell = size_t;
  using Off = size_t;
  double *p;
  Off plane;
  __device__ __forceinline__ StatePtr(const double *q, long nc, int) : p(const_cast<double *>(q)), plane((Off)nc * 8) {}
  template <int AUX = 0>
  __device__ __forceinline__ double load(Off cell8, Off off) const {
    return p[(cell8 + off) >> 3];
  }
  template <int AUX = 0>
  __device__ __forceinline__ void store(double v, Off cell8, Off off) const {
    p[(cell8 + off) >> 3] = v;
  }
};
constexpr int NT = 2;  // non-temporal: data this launch touches once

// the N weights of V variables of one cell, raw (off: byte offset of the first plane)
template <int V, int N, int AUX = 0, class Buf>
__device__ __forceinline__ void load_cell(const Buf &w, typename Buf::Cell cell8, double (&r)[V][N],
                                          typename Buf::Off off = 0) {
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int l = 0; l < N; ++l) {
      r[v][l] = w.template load<AUX>(cell8, off);
      off += w.plane;
    }
}

// Coefficients (by tangential exponent) of the trace of w on the face normal
// to A at xi_A = -1 (S = 0) or +1.
template <int K, int A, int S>
__device__ __forceinline__ void edge_coefs(const double (&w)[(K + 1) * (K + 2) / 2], double (&c)[K + 1]) {
#pragma clang fp contract(off)
  constexpr Line<K> L{};
  static_for<0, K + 1>([&](auto T_) {
    constexpr int t = decltype(T_)::value;
    double x = w[A == 0 ? mode_index<2>(0, t, 0) : mode_index<2>(t, 0, 0)];
    static_for<1, K + 1 - t>([&](auto N_) {
      constexpr int n = decltype(N_)::value;
      constexpr double s = (S == 0 && n % 2 ? -1.0 : 1.0) * L.b[n];
      x = fma(w[A == 0 ? mode_index<2>(n, t, 0) : mode_index<2>(t, n, 0)], s, x);
    });
    c[t] = x;
  });
}

// Coefficients (order of mode_index<2> in the two tangential axes, ascending)
// of the trace of w on the face normal to A at xi_A = -1 (S = 0) or +1.
template <int K, int A, int S>
__device__ __forceinline__ void face_coefs(const double (&w)[(K + 1) * (K + 2) * (K + 3) / 6],
                                  double (&c)[(K + 1) * (K + 2) / 2]) {
#pragma clang fp contract(off)
  constexpr Line<K> L{};
  static_for<0, (K + 1) * (K + 2) / 2>([&](auto J_) {
    constexpr int j = decltype(J_)::value, e1 = mode_exp<2>(j, 0), e2 = mode_exp<2>(j, 1);
    double t = 0.0;
    static_for<0, K + 1>([&](auto N_) {
      constexpr int n = decltype(N_)::value;
      if constexpr (n + e1 + e2 <= K) {
        constexpr int l = A == 0 ? mode_index<3>(n, e1, e2) : A == 1 ? mode_index<3>(e1, n, e2) : mode_index<3>(e1, e2, n);
        constexpr double s = S == 0 && n % 2 ? -1.0 : 1.0;
        if constexpr (n == 0) t = w[l];
        else t = fma(w[l], s * L.b[n], t);
      }
    });
    c[j] = t;
  });
}

// moments m[v][j] = sum_r F_v(x_r) phi_j(x_r) w_r of the HLLC flux over the
// (K+1)^2 face points, from the two traces' coefficients (the low side's
// through cl(v, j): they sit in LDS)
template <int K, int A, int FX, class LO>
__device__ __forceinline__ void face_flux(LO &&cl, const double (&ch)[5][(K + 1) * (K + 2) / 2],
                                 double gamma, double (&m)[5][(K + 1) * (K + 2) / 2]) {
  constexpr int n1 = K + 1, N2 = (K + 1) * (K + 2) / 2;
  const Line<K> &T = line_const<K>();
#pragma unroll
  for (int v = 0; v < 5; ++v)
#pragma unroll
    for (int j = 0; j < N2; ++j) m[v][j] = 0.0;
#pragma unroll 1
  for (int r = 0; r < n1; ++r) {
#pragma clang fp contract(off)
    asm volatile("" ::: "memory");  // the traces in LDS are read again for each row
    double p[n1];
#pragma unroll
    for (int e = 0; e < n1; ++e) p[e] = T.p[r][e];
    const double wr = T.w[r];
    double ul[5][n1], uh[5][n1];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double a[n1], b[n1];
      static_for<0, n1>([&](auto E_) {
        constexpr int e1 = decltype(E_)::value;
        double x = cl(v, mode_index<2>(e1, 0, 0)), y = ch[v][mode_index<2>(e1, 0, 0)];
        static_for<1, n1 - e1>([&](auto G_) {
          constexpr int e2 = decltype(G_)::value;
          x = fma(cl(v, mode_index<2>(e1, e2, 0)), p[e2], x);
          y = fma(ch[v][mode_index<2>(e1, e2, 0)], p[e2], y);
        });
        a[e1] = x;
        b[e1] = y;
      });
      line_values<K, K>(a, ul[v]);
      line_values<K, K>(b, uh[v]);
      DG_FENCE;
    }
    double F[5][n1];
#pragma unroll
    for (int i = 0; i < n1; ++i) {
      const double UL[5] = {ul[0][i], ul[1][i], ul[2][i], ul[3][i], ul[4][i]};
      const double UR[5] = {uh[0][i], uh[1][i], uh[2][i], uh[3][i], uh[4][i]};
      double f[5];
      hllc_line<3, A, FX>(UL, UR, gamma, f);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v][i] = f[v];
      DG_FENCE;
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double s[n1];
      line_moments<K, K>(F[v], s);
      static_for<0, n1>([&](auto E_) {
        constexpr int e1 = decltype(E_)::value;
        static_for<0, n1 - e1>([&](auto G_) {
          constexpr int e2 = decltype(G_)::value;
          m[v][mode_index<2>(e1, e2, 0)] = fma(s[e1], wr * p[e2], m[v][mode_index<2>(e1, e2, 0)]);
        });
      });
      DG_FENCE;
    }
  }
}

// acc_l -+= P~_n(+-1) m_t: the outward flux of side S taken off the accumulators
template <int K, int A, int S>
__device__ __forceinline__ void face_lift(const double (&m)[(K + 1) * (K + 2) / 2],
                                 double (&acc)[(K + 1) * (K + 2) * (K + 3) / 6]) {
  constexpr Line<K> L{};
  static_for<0, (K + 1) * (K + 2) * (K + 3) / 6>([&](auto L_) {
    constexpr int l = decltype(L_)::value, ex = mode_exp<3>(l, 0), ey = mode_exp<3>(l, 1), ez = mode_exp<3>(l, 2);
    constexpr int n = A == 0 ? ex : A == 1 ? ey : ez, e1 = A == 0 ? ey : ex, e2 = A == 2 ? ey : ez;
    constexpr double s = S == 0 ? (n % 2 ? -1.0 : 1.0) : -1.0;  // low side: +F phi(-1), high side: -F phi(+1)
    acc[l] = fma(m[mode_index<2>(e1, e2, 0)], s * L.b[n], acc[l]);
  });
}

}  // namespace dg
