"""GPU: states past the sizes at which addressing or launching changes."""
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _room(gb):
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gb * 2 ** 30:
        pytest.skip(f"needs {gb} GiB of device memory")


def test_limiter_of_a_box_beyond_one_launch():
    """The component limiter takes 256 threads per 64 cells in 2D, so 2^30
    cells are more than one launch holds (2^32 threads).  Slopes in cells of
    the first rows, around the last cell of the first launch and at the end
    are limited to zero (their neighbours' means are equal), the rest of the
    state stays as it is."""
    import torch
    import paper_1506_06140_amd as dg
    print("limiter beyond one launch", flush=True)
    _room(130)
    nx, ny = 32769, 32768
    wl = workloads.workload("blast_amr", dim=2, k=1, n=(nx, ny, 1), refine_lo=(1, 1, 0), refine_hi=(2, 2, 0), limiter=1,
                            positivity=0, mtilde=0.0, length=(nx / 8.0, ny / 8.0, 1.0))
    s = dg.Solver(wl)
    assert s.ncoarse > 2 ** 30
    w = s.empty().zero_()
    coarse, fine = w[:12 * s.ncoarse].view(4, 3, s.ncoarse), w[12 * s.ncoarse:].view(4, 3, s.nfine)
    for b in (coarse, fine):
        b[0, 0] = 1.0
        b[3, 0] = 2.5
    last = 2 ** 30 - 64
    cells = torch.tensor([5 * nx + 7, last - 70, last - 1, last, last + 1, last + 64, s.ncoarse - 5], device="cuda")
    coarse[0, 1, cells] = 0.25
    coarse[3, 2, cells] = -0.125
    s.limit(w)
    assert s.status() == 0
    for v in range(4):
        for l in range(3):
            want = (1.0 if v == 0 else 2.5 if v == 3 else 0.0) if l == 0 else 0.0
            for b in (coarse, fine):
                lo, hi = b[v, l].aminmax()
                assert float(lo) == want and float(hi) == want, (v, l)
    del w, coarse, fine, b, lo, hi, s
    torch.cuda.empty_cache()
