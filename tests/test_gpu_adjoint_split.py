"""GPU: the 2D adjoint kernel that splits a cell's work over four waves, where
its rows of nx + 1 positions meet its blocks of 63 (rows of 61 to 64 cells, two
rows in a block) and where a cell is its own neighbour, with walls and both
wave-speed bounds: <mu, v> against the oracle's complex-step <lam, J v>, to
1e-12 of sum |lam_i (J v)_i| as in the tests of the other sizes, and the stage
against the RHS by its own arithmetic: lam' = acc + lam + dt mu and 2/3 (lam +
dt mu) with three roundings each, so 4 eps of the terms' magnitudes."""
import numpy as np
import pytest

import oracle
from test_gpu_adjoint import _dev, _host, _state, _wl

pytestmark = pytest.mark.gpu

CASES = [
    ("k1_one_row_63", dict(dim=2, k=1, n=(63, 1, 1))),
    ("k1_one_column_walls", dict(dim=2, k=1, n=(1, 65, 1), bc=(1, 1, 0))),
    ("k1_61_davis", dict(dim=2, k=1, n=(61, 3, 1), flux=1)),
    ("k2_62", dict(dim=2, k=2, n=(62, 2, 1))),
    ("k2_64_walls_davis", dict(dim=2, k=2, n=(64, 3, 1), bc=(1, 0, 0), flux=1)),
    ("k2_one_column", dict(dim=2, k=2, n=(1, 33, 1))),
    ("k3_63_walls", dict(dim=2, k=3, n=(63, 2, 1), bc=(0, 1, 0))),
    ("k3_31_davis", dict(dim=2, k=3, n=(31, 5, 1), flux=1)),
    ("k3_125_walls", dict(dim=2, k=3, n=(125, 3, 1), bc=(1, 1, 0))),
]


@pytest.mark.parametrize("case,over", CASES, ids=[c[0] for c in CASES])
def test_adjoint_split(case, over):
    import torch
    import paper_1506_06140_amd as dg
    print("adjoint split", case, flush=True)
    wl = _wl(over)
    o = oracle.Oracle(wl)
    s = dg.Solver(wl)
    rng = np.random.default_rng(7)
    w = _state(o, 5)
    lam = rng.normal(size=o.shape)
    mu = s.adjoint_rhs(_dev(w), _dev(lam))
    for _ in range(3):
        v = rng.normal(size=o.shape)
        _, jv = o.jvp_rhs(w, v)
        assert abs((_host(mu) * v).sum() - (lam * jv).sum()) <= 1e-12 * np.abs(lam * jv).sum()
    l, dt = _dev(lam), torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    acc0 = _dev(rng.normal(size=o.shape))
    eps = 4 * 2.0 ** -52
    size = l.abs() + (dt * mu).abs() + acc0.abs()
    out, acc = s.empty(), acc0.clone()
    s.adjoint_rk_stage(1, dt, _dev(w), l, acc, out, None)
    assert bool(((out - (acc + (l + dt * mu))).abs() <= eps * size).all())
    s.adjoint_rk_stage(3, dt, _dev(w), l, None, out, acc)
    assert bool(((out - 2.0 / 3.0 * (l + dt * mu)).abs() <= eps * size).all())
    assert bool(((acc - l / 3.0).abs() <= eps * size).all())
    s.adjoint_rk_stage(2, dt, _dev(w), l, acc0, out, acc0.copy_(acc))
    assert bool(((out - 0.25 * (l + dt * mu)).abs() <= eps * size).all())
    assert bool(((acc0 - (acc + 0.75 * l)).abs() <= eps * size).all())
