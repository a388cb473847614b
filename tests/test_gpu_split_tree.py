"""GPU: the quadtree stage kernel (five waves per 64 leaves) against the FP64
oracle at leaf counts around its blocks and with every face kind: no
refinement on 63, 64 and 65 leaves, random refinement by one and two levels,
walls, both wave-speed bounds.  The RHS to 1e-12 of fac(|V| + |S|) and per
element of the summands (a hanging side has 2 (k + 1) points: about 150 terms,
3e-14), a stage with an earlier state to 1e-12."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs_modes, check_state_modes

pytestmark = pytest.mark.gpu

CASES = [
    ("k1_63_flat", 1, (7, 9), 0, {}),
    ("k2_64_flat_walls", 2, (8, 8), 0, dict(bc=(1, 1, 0))),
    ("k3_65_flat", 3, (13, 5), 0, dict(flux=1)),
    ("k1_two_levels_walls", 1, (6, 5), 2, dict(bc=(1, 0, 0))),
    ("k2_two_levels", 2, (6, 6), 2, dict(flux=1)),
    ("k3_one_level", 3, (5, 7), 1, {}),
    ("k3_two_levels_walls", 3, (6, 5), 2, dict(bc=(0, 1, 0))),
]


@pytest.mark.parametrize("case,k,n,levels,over", CASES, ids=[c[0] for c in CASES])
def test_tree_stage_matches_oracle(case, k, n, levels, over):
    import torch
    import paper_1506_06140_amd as dg
    print("split tree", case, flush=True)
    wl = workloads.workload("kh2d", k=k, n=(n[0], n[1], 1), length=(n[0] / 8, n[1] / 8, 1.0), limiter=0, positivity=0,
                            rk="rk3", **over)
    bc = wl["bc"]
    leaves = workloads.random_tree(n, levels, 0.4, 11, periodic=(not bc[0], not bc[1]))
    o = oracle.TreeOracle(wl, leaves)
    r = np.random.default_rng(5)
    shape = (4, (k + 1) * (k + 2) // 2, len(leaves))
    w, u = (0.02 * r.uniform(-1, 1, size=shape) for _ in range(2))
    for x in (w, u):
        rho = 1.0 + 0.2 * r.uniform(-1, 1, size=shape[2])
        vx, vy = (0.3 * r.uniform(-1, 1, size=shape[2]) + b for b in (0.4, -0.3))
        x[:, 0] = rho, rho * vx, rho * vy, (1.0 + 0.2 * r.uniform(-1, 1, size=shape[2])) / 0.4 + 0.5 * rho * (vx ** 2 + vy ** 2)
    s = dg.TreeSolver(wl, leaves)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    V, S, A = (np.asarray(x).reshape(shape) for x in o.terms(w))
    check_rhs_modes(s.rhs(dev(w)).cpu().numpy().reshape(shape), V, S, A, f"{case} rhs")
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    got = s.rk_stage(2, dt, dev(u), dev(w)).cpu().numpy().reshape(shape)
    check_state_modes(got, np.asarray(o.rk3_stage(2, 1e-3, u, w)).reshape(shape), f"{case} stage 2")
    assert s.status() == 0
