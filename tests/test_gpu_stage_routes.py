"""GPU: FP64 stages on both sides of the choice between the sum-factorised
kernels and the others, against the FP64 oracle: grids and boxes that are
narrow in x or in x and y (one thread per cell, MFMA), and ones with several
planes a workgroup of the four-wave kernel together with walls and both
wave-speed bounds.  The RHS to 1e-12 of fac(|V| + |S|), the stages to 1e-12.
Each case states which side it is on."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs, check_rhs_modes
from test_gpu_march import _state
from test_gpu_split3d import _dev, _stages
from test_stage_rules import choices

pytestmark = pytest.mark.gpu

GRIDS = [  # k, grid, sum-factorised, options
    (1, (2, 180, 180), False, dict(bc=(1, 0, 0))),
    (2, (1, 160, 160), False, dict(bc=(0, 1, 0), flux=1)),
    (3, (9, 14, 99), False, dict(bc=(1, 1, 0), flux=1)),
    (3, (4, 4, 1100), False, dict(bc=(0, 0, 1))),
    (3, (9, 36, 52), True, dict(bc=(1, 1, 0), flux=1)),
]
BOXES = [
    (2, (3, 3, 300), ((1, 1, 1), (2, 2, 299)), False, dict(bc=(1, 1, 1))),
    (3, (3, 3, 300), ((1, 1, 1), (2, 2, 299)), False, dict(flux=1)),
    (2, (12, 12, 40), ((1, 1, 1), (11, 11, 39)), True, dict(bc=(1, 1, 1))),
    (2, (16, 16, 16), ((7, 7, 7), (8, 8, 8)), True, dict(flux=1)),  # a fine block of a few cells at the state's end
    (3, (8, 8, 40), ((1, 1, 1), (7, 7, 39)), True, dict(bc=(0, 1, 1), flux=1)),
]


def box_state(o, seed):
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


@pytest.mark.parametrize("k,n,factorised,over", GRIDS)
def test_grids(k, n, factorised, over, tmp_path):
    import paper_1506_06140_amd as dg
    print("route", k, n, flush=True)
    assert choices(tmp_path, [(k, n, None)]) == [factorised]
    wl = workloads.workload("kh3d", k=k, n=n, limiter=0, positivity=0, length=tuple(m / n[0] for m in n), **over)
    o = oracle.Oracle(wl)
    w, u = _state(o, 1), _state(o, 2)
    s = dg.Solver(wl)
    V, S, A = o.terms_cells(w, with_abs=True)
    check_rhs_modes(s.rhs(_dev(w)).cpu().numpy().reshape(V.shape), V, S, A, f"{n} rhs")
    _stages(s, o, w, u, f"{n}")


@pytest.mark.parametrize("k,n,box,factorised,over", BOXES)
def test_boxes(k, n, box, factorised, over, tmp_path):
    import paper_1506_06140_amd as dg
    print("route box", k, n, box, flush=True)
    assert choices(tmp_path, [(k, n, box)]) == [factorised]
    wl = workloads.workload("blast_amr", dim=3, k=k, n=n, refine_lo=box[0], refine_hi=box[1], limiter=0, positivity=0,
                            length=tuple(m / 8.0 for m in n), **over)
    o = oracle.AmrOracle(wl)
    w, u = box_state(o, 1), box_state(o, 2)
    s = dg.Solver(wl)
    V, S, A = o.terms_cells(w, with_abs=True)
    check_rhs(o, s.rhs(_dev(w)).cpu().numpy(), V, S, A, f"{n} {box} rhs")
    _stages(s, o, w, u, f"{n} {box}")


@pytest.mark.parametrize("ny,flux,bc", [(24192, 0, 0), (24193, 1, 0), (24500, 0, 1)])
def test_adjoint_of_one_cell_rows(ny, flux, bc):
    """Both sides of the 2D adjoint's choice at k = 3 (768 workgroups of 63
    positions, two a cell): <mu, v> against the oracle's <lam, J v> to 1e-12 of
    sum |lam_i (J v)_i|."""
    import paper_1506_06140_amd as dg
    from test_gpu_adjoint import _dev as dev, _state as state, _wl
    print("route adjoint", ny, flux, bc, flush=True)
    wl = _wl(dict(dim=2, k=3, n=(1, ny, 1), flux=flux, bc=(bc, bc, 0)))
    o = oracle.Oracle(wl)
    s = dg.Solver(wl)
    rng = np.random.default_rng(7)
    w, lam, v = state(o, 5), rng.normal(size=o.shape), rng.normal(size=o.shape)
    mu = s.adjoint_rhs(dev(w), dev(lam)).cpu().numpy()
    _, jv = o.jvp_rhs(w, v)
    assert abs((mu * v).sum() - (lam * jv).sum()) <= 1e-12 * np.abs(lam * jv).sum()
    assert s.status() == 0
