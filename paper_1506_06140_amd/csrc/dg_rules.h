// Rules on sizes alone (host only): how many items a launch takes, and which
// FP64 kernel 3D stages and the 2D adjoint run on.
#pragma once

namespace dg {

// Items that one launch may take of a kernel whose workgroups of `threads` take
// 64 each: a launch holds fewer than 2^32 threads along a dimension, which
// workgroups of several threads an item reach before the grids' 2^31 cells do.
constexpr long launch_items(long threads) { return ((1L << 32) - 1) / threads * 64; }

constexpr long kCusPerGpu = 256;            // MI355X
constexpr long kSimdsPerGpu = 4 * kCusPerGpu;

// Waves of k_rhs_march3d that run at once: two per SIMD at k = 1, one at k = 2.
constexpr long march_slots(int k) { return k == 1 ? 2 * kSimdsPerGpu : kSimdsPerGpu; }

// Planes per wave: all waves run alike, one (k = 2) or two (k = 1) per SIMD at
// a time, and a wave's cost is about its planes plus a quarter (the first
// face, the first loads).  128^3, k = 2, us per launch for 4, 7, 8, 12, 16, 32
// planes: 1366, 1346, 1423, 1330, 1647, 2164; k = 1: 448, 444, 453, 448, 500,
// 609; 64^3, k = 1, for 1, 3, 6, 12 planes: 87, 79, 85, 150.
inline int march_len(long columns, int nz, long slots) {
  double best = 0.0;
  int at = 1;
  for (int len = 1; len <= nz && len <= 64; ++len) {
    const long waves = (columns * ((nz + len - 1) / len) + 61) / 62;
    const double cost = (double)((waves + slots - 1) / slots) * (len + 0.25);
    if (len == 1 || cost < best) {
      best = cost;
      at = len;
    }
  }
  return at;
}

// k_rhs_march3d on uniform grids at k = 1 and 2, against k_rhs_stage (k = 1)
// and the MFMA kernel (k = 2).  Two exceptions:
// at k = 2 a grid of at most one 64-cell block per compute unit stays on the
// MFMA kernel, whose 16-cell waves finish sooner when the chip is not full (us
// per launch, MFMA against march: 16^3 27.8, 39.1; 25 x 25 x 26 36.5, 43; 26^3
// 55.2, 43.6; 32^3 57.4, 48.2; 64 x 9 x 100 101, 61);
// of a march's lanes nx / (nx + 2) are real, so grids of narrow rows stay on
// the other kernel once they need more than one plane a wave: rows of one or
// two cells at k = 1 (other kernel, march: 1 x 200 x 200 below the line, 1 x 357
// x 358 49, 85; 1 x 707 x 707 171, 273; 2 x 180 x 180 40, 47; 2 x 500 x 500 161,
// 183; 3 x 408 x 408 165, 165), of one cell at k = 2 (1 x 158 x 158 55, 81; 1 x 400
// x 400 214, 287; rows of two cells within 7 % either way: 2 x 200 x 200 115, 121;
// 2 x 400 x 400 433, 394).
inline bool march3d_faster(int k, long nx, long ny, long nz) {
  if (k == 2 && nx * ny * nz <= 64 * kCusPerGpu) return false;
  return nx > (k == 1 ? 2 : 1) || ((nx + 2) * ny * nz + 61) / 62 <= march_slots(k);
}

// k_rhs_split3d's work: (63-column block, plane) pairs of one block of cells,
// in equal runs on kCusPerGpu workgroups.
inline long split_planes(long nx, long ny, long nz) { return ((nx + 1) * ny + 62) / 63 * nz; }
inline long rounds(long n, long per) { return (n + per - 1) / per; }

// k_rhs_split3d against the MFMA kernel, both by the time of their longest
// workgroup (us).  A run of planes costs a plane 36 and a column start 12 (the
// z face below it); the MFMA kernel takes 67 for every 64 cells a compute
// unit, 85 if that is all.  The split kernel's lanes hold whole rows of one
// z plane, so grids that are narrow in x and y leave most of them idle.  Of 130
// grids timed on both kernels the rule's choice was at worst 3 % the slower
// one (us, MFMA against split: 32^3 135, 137; 26^3 135, 89; 62 x 47 x 48 628, 347;
// 3 x 64 x 64 91, 101; 2 x 128 x 128 137, 167; 2 x 160 x 160 253, 191; 8 x 8 x
// 1000 262, 287; 4 x 4 x 2000 138, 279; 1 x 1 x 40000 204, 5027).
inline bool split3d_faster(long nx, long ny, long nz) {
  const long run = rounds(split_planes(nx, ny, nz), kCusPerGpu);
  const long r = rounds(nx * ny * nz, 64 * kCusPerGpu);
  return 8 + 36 * run + 12 * rounds(run, nz) <= (r == 1 ? 85 : 67.5 * r);
}

// The same on the refined box (base grid n, fine block nf) at k = 2 and 3,
// both kernels with their hanging faces; those cost the MFMA kernel more where
// a wave's 16 cells of the fine block span whole rows.  Of 100 boxes timed on
// both, the choice was at worst 9 % the slower one (us, MFMA against split: k =
// 2, 20^3 with 10^3 refined 76, 66; 3 x 3 x 1000 112, 260; 8 x 8 x 300 155, 175;
// k = 3, 20^3 with 10^3 refined 112, 128; 28^3 with 14^3 230, 184; 48 x 8 x 32 with
// 27 x 3 x 6 99, 144; 3 x 3 x 1000 182, 494; 3 x 34 x 34 148, 138).
inline bool split3d_box_faster(int k, const long n[3], const long nf[3]) {
  const long run = rounds(split_planes(n[0], n[1], n[2]) + split_planes(nf[0], nf[1], nf[2]), kCusPerGpu);
  const long r = rounds(rounds(n[0] * n[1] * n[2], 64) + rounds(nf[0] * nf[1] * nf[2], 64), kCusPerGpu);
  const bool thin = nf[0] < 16;
  return k == 2 ? 30 + 20 * run <= 47 + 25 * r + (thin ? 20 : 0) : 42 + 41 * run <= 45 + 70 * r + (thin ? 30 : 0);
}

// k_adjoint_split2d against k_adjoint_quad2d (four lanes per cell): the former's
// rows of nx + 1 positions are half idle at nx = 1, which at k = 3 costs more
// than the split gains from three workgroups a compute unit on (us a stage, quad
// against split: 1 x 8192 31, 21; 1 x 24000 41, 38; 1 x 32768 42, 53; 1 x 524288
// 613, 765; 2 x 65536 145, 130; k = 2, 1 x 524288 397, 359).
inline bool adjoint_split_faster(int k, long nx, long ny) {
  return k < 3 || nx > 1 || rounds((nx + 1) * ny, 63) <= 3 * kCusPerGpu;
}

}  // namespace dg
