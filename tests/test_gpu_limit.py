"""GPU: the component-wise limiter with one wave per variable (refined boxes,
3D uniform grids at k = 2) against the FP64 oracle where its blocks of 64
cells end and where a neighbour mean is not a cell's: 63, 64, 65 and 1 cells,
walls, a box of one coarse cell, boxes a cell from the domain's faces and two
cells apart across the periodic wrap.  Rough states, so that some variables
of some cells are limited and others not.  The limiter's arithmetic is a few
operations per value: states to 1e-12 (check_state)."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_state
from test_gpu_amr import _wl, rough_amr_state
from test_gpu_march import _state

pytestmark = pytest.mark.gpu

GRIDS = [((1, 1, 1), 0), ((63, 1, 1), 1), ((4, 4, 4), 0), ((13, 5, 1), 1), ((9, 8, 7), 0)]
BOXES = [
    ("2d_k1_one_cell", dict(dim=2, k=1, n=(3, 3, 1), lo=(1, 1, 0), hi=(2, 2, 0))),
    ("2d_k3_edges", dict(dim=2, k=3, n=(33, 6, 1), lo=(1, 1, 0), hi=(32, 5, 0))),
    ("3d_k1_flat", dict(dim=3, k=1, n=(8, 4, 3), lo=(1, 1, 1), hi=(7, 3, 2))),
    ("3d_k2_one_cell", dict(dim=3, k=2, n=(3, 4, 5), lo=(1, 2, 3), hi=(2, 3, 4))),
    ("3d_k3_walls", dict(dim=3, k=3, n=(5, 4, 4), lo=(1, 1, 1), hi=(4, 3, 3), bc=(1, 1, 1))),
]


def _check(o, s, w, case):
    import torch
    ref, st = o.limit(w.copy())
    assert st == 0
    d = torch.from_numpy(np.ascontiguousarray(w)).cuda()
    s.limit(d)
    check_state(o, d.cpu().numpy(), ref, case)
    assert s.status() == 0


@pytest.mark.parametrize("positivity", [0, 1])
@pytest.mark.parametrize("n,bc", GRIDS)
def test_limit_uniform(n, bc, positivity):
    import paper_1506_06140_amd as dg
    print("limit", n, bc, positivity, flush=True)
    wl = workloads.workload("kh3d", k=2, n=n, length=tuple(m / n[0] for m in n), bc=(bc,) * 3, limiter=1,
                            positivity=positivity)
    o = oracle.Oracle(wl)
    _check(o, dg.Solver(wl), _state(o, 3), f"limit {n}")


@pytest.mark.parametrize("case,spec", BOXES, ids=[c[0] for c in BOXES])
def test_limit_box(case, spec):
    import paper_1506_06140_amd as dg
    print("limit box", case, flush=True)
    wl = _wl(**spec, ic="kh3d")
    o = oracle.AmrOracle(wl)
    _check(o, dg.Solver(wl), rough_amr_state(o, 5), f"limit box {case}")
