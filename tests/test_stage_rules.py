"""CPU: the choice between the FP64 stage kernels, compiled for the host and
checked against launches timed on both kernels (us: the one it may replace, the
sum-factorised one), a tenth of slack for shapes where the two are close."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1506_06140_amd", "csrc")

MAIN = """
#include "dg_rules.h"
#include <cstdio>
int main() {
  int k, box;
  long n[6];
  while (scanf("%d %d %ld %ld %ld %ld %ld %ld", &k, &box, n, n + 1, n + 2, n + 3, n + 4, n + 5) == 8)
    printf("%d\\n", box == 2 ? (int)dg::adjoint_split_faster(k, n[0], n[1])
                   : box   ? (int)dg::split3d_box_faster(k, n, n + 3)
                   : k < 3 ? (int)dg::march3d_faster(k, n[0], n[1], n[2])
                           : (int)dg::split3d_faster(n[0], n[1], n[2]));
}
"""

# (k, grid, refined box or None, other kernel, sum-factorised kernel)
TIMED = [
    # one-thread-per-cell kernel against the march along z, k = 1
    (1, (1, 16, 16), None, 28.7, 17.0), (1, (1, 200, 200), None, 31.5, 30.2), (1, (1, 357, 358), None, 49.3, 85.3),
    (1, (1, 707, 707), None, 170.7, 272.7), (1, (2, 128, 128), None, 30.7, 28.2), (1, (2, 180, 180), None, 40.3, 47.2),
    (1, (2, 500, 500), None, 160.7, 183.2), (1, (3, 408, 408), None, 165.0, 165.2), (1, (4, 256, 256), None, 97.9, 93.9),
    (1, (300000, 1, 1), None, 101.1, 65.7), (1, (128, 128, 128), None, 681.0, 421.0),
    # MFMA kernel against the march, k = 2
    (2, (16, 16, 16), None, 27.8, 39.1), (2, (26, 26, 26), None, 55.2, 43.6), (2, (1, 158, 158), None, 54.5, 80.6),
    (2, (1, 400, 400), None, 214.3, 287.0), (2, (2, 200, 200), None, 115.4, 121.0), (2, (3, 300, 300), None, 366.0, 290.3),
    (2, (256, 256, 1), None, 95.7, 84.7), (2, (128, 128, 128), None, 2695.0, 1299.0),
    # MFMA kernel against the split over four waves, k = 3
    (3, (8, 8, 8), None, 67.0, 52.0), (3, (3, 64, 64), None, 91.0, 101.0), (3, (24, 24, 24), None, 96.0, 60.0),
    (3, (26, 26, 26), None, 134.6, 88.7), (3, (32, 32, 32), None, 135.4, 136.5), (3, (2, 128, 128), None, 136.9, 166.9),
    (3, (2, 160, 160), None, 252.8, 191.2), (3, (1, 288, 288), None, 381.6, 423.8), (3, (1, 1, 40000), None, 203.5, 5026.6),
    (3, (4, 4, 2000), None, 138.2, 278.8), (3, (8, 8, 1000), None, 261.5, 286.7), (3, (2, 4, 19880), None, 687.7, 2589.3),
    (3, (8, 7, 2859), None, 695.2, 436.8), (3, (40000, 1, 1), None, 202.8, 155.9), (3, (256, 256, 1), None, 264.7, 255.1),
    (3, (62, 47, 48), None, 628.4, 346.7), (3, (64, 64, 64), None, 1107.0, 629.0),
    # refined boxes
    (2, (3, 3, 3), ((1, 1, 1), (2, 2, 2)), 78.4, 43.3), (2, (3, 3, 1000), ((1, 1, 1), (2, 2, 999)), 111.7, 259.5),
    (2, (3, 34, 34), ((1, 1, 1), (2, 33, 33)), 93.8, 74.8), (2, (8, 8, 300), ((2, 2, 1), (6, 6, 299)), 155.3, 174.6),
    (2, (20, 20, 20), ((5, 5, 5), (15, 15, 15)), 75.5, 66.3), (2, (4, 3, 400), ((1, 1, 7), (3, 2, 192)), 84.8, 100.1),
    (2, (1000, 3, 3), ((1, 1, 1), (999, 2, 2)), 68.1, 73.9), (2, (48, 48, 48), ((12, 12, 12), (36, 36, 36)), 422.0, 324.0),
    (3, (3, 3, 1000), ((1, 1, 1), (2, 2, 999)), 181.9, 494.4), (3, (16, 16, 16), ((4, 4, 4), (12, 12, 12)), 107.7, 83.1),
    (3, (20, 20, 20), ((5, 5, 5), (15, 15, 15)), 111.9, 128.2), (3, (3, 34, 34), ((1, 1, 1), (2, 33, 33)), 148.0, 138.4),
    (3, (48, 8, 32), ((8, 1, 4), (35, 4, 10)), 98.9, 143.7), (3, (28, 28, 28), ((7, 7, 7), (21, 21, 21)), 230.1, 183.7),
    (3, (64, 64, 64), ((16, 16, 16), (48, 48, 48)), 2469.0, 1440.0),
    # 2D adjoint: four lanes per cell against the split over four waves
    (1, (1, 524288, 1), "adjoint", 229.1, 186.4), (2, (1, 524288, 1), "adjoint", 396.7, 359.2),
    (3, (1, 8192, 1), "adjoint", 30.8, 21.4), (3, (1, 24000, 1), "adjoint", 41.1, 37.8),
    (3, (1, 32768, 1), "adjoint", 41.7, 52.7), (3, (1, 524288, 1), "adjoint", 613.2, 765.4),
    (3, (2, 65536, 1), "adjoint", 145.2, 130.0), (3, (512, 512, 1), "adjoint", 320.0, 248.0),
]


def choices(work, cases):
    """For each (k, grid, box or None, ...): whether the sum-factorised kernel is chosen."""
    (work / "rules.cpp").write_text(MAIN)
    exe = str(work / "rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(work / "rules.cpp")], check=True)
    rows = []
    for k, n, box, *_ in cases:
        nf = [2 * (h - l) for l, h in zip(*box)] if box and box != "adjoint" else [0, 0, 0]
        rows.append(" ".join(str(x) for x in (k, 2 if box == "adjoint" else int(box is not None), *n, *nf)))
    out = subprocess.run([exe], input="\n".join(rows), capture_output=True, text=True, check=True).stdout.split()
    return [bool(int(x)) for x in out]


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    return choices(tmp_path_factory.mktemp("rules"), TIMED)


def test_a_launch_holds_less_than_2_to_the_32_threads(tmp_path):
    (tmp_path / "items.cpp").write_text("""
#include "dg_rules.h"
constexpr bool fits(long threads) {
  const long n = dg::launch_items(threads);
  return n % 64 == 0 && n / 64 * threads < (1L << 32) && (n / 64 + 1) * threads >= (1L << 32);
}
static_assert(fits(256) && fits(320), "the most whole workgroups below 2^32 threads");
""")
    subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", CSRC, str(tmp_path / "items.cpp")], check=True)


@pytest.mark.parametrize("i", range(len(TIMED)), ids=["k%d_%s%s" % (t[0], "x".join(map(str, t[1])), "_adjoint" if t[2] == "adjoint" else "_box" if t[2] else "")
                                                      for t in TIMED])
def test_the_faster_kernel_is_chosen(chosen, i):
    other, factorised = TIMED[i][3:]
    assert (factorised if chosen[i] else other) <= 1.1 * min(other, factorised)
