"""GPU: the sum-factorised 3D stage kernel (k = 1, and k = 2 on grids of more
than one 64-cell block per compute unit) against the FP64 oracle where its
work split can go wrong: rows of 62 +- 1 cells and columns that cross a wave,
a last run of planes shorter than the others, one cell per axis, walls on
every axis and both wave-speed bounds.  The RHS to 1e-12 of fac(|V| + |S|) and
per element of the summands (the bound of a sum of about 200 rounded terms is
4e-14), stages with one and with several earlier states to 1e-12."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs_modes, check_state

pytestmark = pytest.mark.gpu

CASES = [
    ("k1_one_cell_rows", dict(k=1, n=(1, 3, 2))),
    ("k1_62_walls", dict(k=1, n=(62, 5, 7), bc=(1, 1, 1))),
    ("k1_61_davis", dict(k=1, n=(61, 4, 9), flux=1, bc=(0, 1, 0))),
    ("k1_130_long", dict(k=1, n=(130, 9, 31), bc=(1, 0, 0))),
    ("k2_61_periodic", dict(k=2, n=(61, 17, 16))),
    ("k2_63_walls", dict(k=2, n=(63, 9, 31), bc=(1, 1, 1))),
    ("k2_9_davis", dict(k=2, n=(9, 43, 47), flux=1, bc=(0, 0, 1))),
]


def _state(o, seed):
    """Means around (1, 0.4, -0.3, 0.2; p = 1) and modes of a few per cent."""
    r = np.random.default_rng(seed)
    w = 0.02 * r.uniform(-1, 1, size=o.shape)
    c = o.shape[2:]
    rho = 1.0 + 0.2 * r.uniform(-1, 1, size=c)
    vel = [b + 0.3 * r.uniform(-1, 1, size=c) for b in (0.4, -0.3, 0.2)]
    w[0, 0] = rho
    for a in range(3):
        w[1 + a, 0] = rho * vel[a]
    w[4, 0] = (1.0 + 0.2 * r.uniform(-1, 1, size=c)) / 0.4 + 0.5 * rho * sum(v * v for v in vel)
    return w


@pytest.mark.parametrize("case,spec", CASES, ids=[c[0] for c in CASES])
def test_march_matches_oracle(case, spec):
    import torch
    import paper_1506_06140_amd as dg
    print("march", case, flush=True)
    n = spec["n"]
    wl = workloads.workload("kh3d", limiter=0, positivity=0, length=tuple(m / n[0] for m in n), **spec)
    o = oracle.Oracle(wl)
    w, u = _state(o, 1), _state(o, 2)
    s = dg.Solver(wl)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    V, S, A = o.terms_cells(w, with_abs=True)
    L = s.rhs(dev(w)).cpu().numpy()
    check_rhs_modes(L.reshape(V.shape), V, S, A, f"{case} rhs")
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    for stage, wn in ((1, None), (2, u), (3, u)):
        got = s.rk_stage(stage, dt, None if wn is None else dev(wn), dev(w)).cpu().numpy()
        check_state(o, got, o.rk3_stage(stage, 1e-3, u, w), f"{case} stage {stage}")
    # the fifth stage of RK_4 takes four earlier states
    tab = dg.TABLEAUS["rk4"]
    s.set_tableau(*tab)
    ys = [_state(o, 3 + j) for j in range(5)]
    got = s.tableau_stage(5, dt, [dev(y) for y in ys]).cpu().numpy()
    a = np.array(tab[0]).reshape(5, 5)
    check_state(o, got, o.tableau_stage(a, np.array(tab[1]), 5, 1e-3, ys), f"{case} tableau stage")
    assert s.status() == 0
