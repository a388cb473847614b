"""GPU: the 3D stage kernel that splits 63 cells' work over four waves (k = 3,
and the refined box at k = 2, 3) against the FP64 oracle where its split can
go wrong: rows of 62 to 64 cells and of one cell, columns that start in the
middle of a workgroup's planes (more planes than workgroups), walls on every
axis, both wave-speed bounds; boxes of one coarse cell, of a whole row's
width, and with rows that cross a wave.  The RHS to 1e-12 of fac(|V| + |S|)
(a sum of about 500 rounded terms: 1e-13), the stages to 1e-12."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs, check_rhs_modes, check_state
from test_gpu_march import _state

pytestmark = pytest.mark.gpu

GRIDS = [
    ("one_cell", dict(n=(1, 1, 1))),
    ("one_cell_rows_walls", dict(n=(1, 5, 3), bc=(1, 1, 1))),
    ("62_walls", dict(n=(62, 3, 4), bc=(1, 0, 1))),
    ("63_davis", dict(n=(63, 2, 3), flux=1, bc=(0, 1, 0))),
    ("64_long", dict(n=(64, 2, 131))),
    ("9_walls_davis", dict(n=(9, 14, 99), flux=1, bc=(1, 1, 0))),
]
BOXES = [
    ("k2_one_coarse_cell", dict(k=2, n=(3, 3, 3), lo=(1, 1, 1), hi=(2, 2, 2))),
    ("k2_wide_walls", dict(k=2, n=(66, 5, 4), lo=(1, 2, 1), hi=(65, 3, 3), bc=(1, 1, 1))),
    ("k3_flat_davis", dict(k=3, n=(7, 9, 5), lo=(2, 1, 3), hi=(6, 8, 4), flux=1)),
    ("k3_wide", dict(k=3, n=(36, 5, 5), lo=(2, 1, 2), hi=(34, 4, 4))),
]
dt0 = 1e-3


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _stages(s, o, w, u, case):
    import torch
    dt = torch.full((1,), dt0, dtype=torch.float64, device="cuda")
    for stage, wn in ((1, None), (2, u), (3, u)):
        got = s.rk_stage(stage, dt, None if wn is None else _dev(wn), _dev(w)).cpu().numpy()
        check_state(o, got, o.rk3_stage(stage, dt0, u, w), f"{case} stage {stage}")
    assert s.status() == 0


@pytest.mark.parametrize("case,spec", GRIDS, ids=[c[0] for c in GRIDS])
def test_split3d_matches_oracle(case, spec):
    import torch
    import paper_1506_06140_amd as dg
    print("split3d", case, flush=True)
    n = spec["n"]
    wl = workloads.workload("kh3d", k=3, limiter=0, positivity=0, length=tuple(m / n[0] for m in n), **spec)
    o = oracle.Oracle(wl)
    w, u = _state(o, 1), _state(o, 2)
    s = dg.Solver(wl)
    V, S, A = o.terms_cells(w, with_abs=True)
    check_rhs_modes(s.rhs(_dev(w)).cpu().numpy().reshape(V.shape), V, S, A, f"{case} rhs")
    _stages(s, o, w, u, case)
    # the fifth stage of RK_4 takes four earlier states
    tab = dg.TABLEAUS["rk4"]
    s.set_tableau(*tab)
    dt = torch.full((1,), dt0, dtype=torch.float64, device="cuda")
    ys = [_state(o, 3 + j) for j in range(5)]
    got = s.tableau_stage(5, dt, [_dev(y) for y in ys]).cpu().numpy()
    a = np.array(tab[0]).reshape(5, 5)
    check_state(o, got, o.tableau_stage(a, np.array(tab[1]), 5, dt0, ys), f"{case} tableau stage")


@pytest.mark.parametrize("case,spec", BOXES, ids=[c[0] for c in BOXES])
def test_split3d_box_matches_oracle(case, spec):
    import paper_1506_06140_amd as dg
    print("split3d box", case, flush=True)
    spec = dict(spec)
    wl = workloads.workload("blast_amr", dim=3, refine_lo=spec.pop("lo"), refine_hi=spec.pop("hi"), limiter=0,
                            positivity=0, length=tuple(m / 8.0 for m in spec["n"]), **spec)
    o = oracle.AmrOracle(wl)

    def state(seed):
        r = np.random.default_rng(seed)
        w = o.initial_state()
        for b in o.blocks(w):  # views into w
            b[:, 1:] = 0.02 * r.uniform(-1, 1, size=b[:, 1:].shape)
            rho = 1.0 + 0.2 * r.uniform(-1, 1, size=b[0, 0].shape)
            vel = [c + 0.3 * r.uniform(-1, 1, size=rho.shape) for c in (0.4, -0.3, 0.2)]
            b[0, 0] = rho
            for a in range(3):
                b[1 + a, 0] = rho * vel[a]
            b[4, 0] = (1.0 + 0.2 * r.uniform(-1, 1, size=rho.shape)) / 0.4 + 0.5 * rho * sum(v * v for v in vel)
        return w

    w, u = state(1), state(2)
    s = dg.Solver(wl)
    V, S, A = o.terms_cells(w, with_abs=True)
    check_rhs(o, s.rhs(_dev(w)).cpu().numpy(), V, S, A, f"{case} rhs")
    _stages(s, o, w, u, case)
