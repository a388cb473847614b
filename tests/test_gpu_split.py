"""GPU: the 2D stage kernel that splits a cell's work over four waves, against
the FP64 oracle where its rows of nx + 1 positions meet its blocks of 63: rows
of 61 to 64 cells, one-cell rows and columns, walls, both wave-speed bounds,
gravity, k = 1..4.  The RHS to 1e-12 of fac(|V| + |S|) and per element of the
summands (at most about 100 rounded terms: 2e-14), two one-call steps to 1e-12
and their dt to 1e-14."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs_modes, check_state

pytestmark = pytest.mark.gpu

CASES = [
    ("k1_one_row", dict(name="density_wave", k=1, n=(63, 1, 1))),
    ("k1_one_column_walls", dict(name="density_wave", k=1, n=(1, 64, 1), bc=(1, 1, 0))),
    ("k1_62_rk4", dict(name="density_wave", k=1, n=(62, 5, 1), rk="rk4")),
    ("k2_64_walls", dict(name="density_wave", k=2, n=(64, 9, 1), bc=(1, 0, 0))),
    ("k2_61_davis", dict(name="density_wave", k=2, n=(61, 33, 1), bc=(0, 1, 0), flux=1, rk="rk2")),
    ("k3_63", dict(name="density_wave", k=3, n=(63, 3, 1))),
    ("k3_125_walls", dict(name="density_wave", k=3, n=(125, 7, 1), bc=(1, 1, 0), rk="rk4")),
    ("k4_62_davis", dict(name="density_wave", k=4, n=(62, 4, 1), flux=1)),
    ("k4_65_walls", dict(name="density_wave", k=4, n=(65, 6, 1), bc=(1, 1, 0), rk="rk4")),
    ("k2_gravity", dict(name="kepler", k=2, n=(63, 21, 1), rk="rk3")),
    ("k3_gravity", dict(name="kepler", k=3, n=(31, 62, 1), rk="rk2")),
]


@pytest.mark.parametrize("case,spec", CASES, ids=[c[0] for c in CASES])
def test_split_matches_oracle(case, spec):
    import torch
    import paper_1506_06140_amd as dg
    print("split", case, flush=True)
    spec = dict(spec)
    n, size = spec["n"], 6.0 if spec["name"] == "kepler" else 1.0
    wl = workloads.workload(spec.pop("name"), length=(size, size * n[1] / n[0], size), **spec)
    o = oracle.Oracle(wl)
    w0 = o.initial_state()
    if wl["positivity"]:
        w0, st = o.limit(w0)
        assert st == 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    s = dg.Solver(wl)
    L = s.rhs(dev(w0)).cpu().numpy()
    if wl["gravity"] is None:
        V, S, A = o.terms_cells(w0, with_abs=True)
        check_rhs_modes(L.reshape(V.shape), V, S, A, f"{case} rhs")
    else:
        check_state(o, L, o.rhs(w0), f"{case} rhs")
    bufs = [s.empty() for _ in range(s.stages)]
    dt, rate = s.scalar(), s.rate_state()
    w, ref = dev(w0), w0
    s.max_rate(w, rate)
    for i in range(2):
        ref, dt_ref = o.step(ref)
        w = s.rk_step(w, bufs, dt, rate).clone()
        assert float(dt.cpu()[0]) == pytest.approx(dt_ref, rel=1e-14)
        check_state(o, w.cpu().numpy(), ref, f"{case} step {i}")
    assert s.status() == 0
