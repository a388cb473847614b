"""GPU: the limiters on states that they change in part, against the FP64
oracle, at the sizes where the component limiter's blocks of 64 cells end and
where a neighbour's mean is not a cell's.  Slopes are drawn around the TVB
bound mtilde dx (up to 1.3 times it, so each axis is limited in about a quarter
of the variables), and a third of the cells is thin (means of 2 %), so that
their points go negative.  Each case checks on the oracle's result, for each
block of cells by itself, that some variables and not all are limited and that
the positivity pass scales some cells and not all; states to 1e-12."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_state

pytestmark = pytest.mark.gpu

GRIDS = [  # dim, k, grid, walls
    (3, 2, (63, 1, 1), 1), (3, 2, (4, 4, 4), 0), (3, 2, (13, 5, 1), 1), (3, 2, (9, 8, 7), 0), (3, 1, (5, 9, 7), 1),
    (3, 3, (7, 4, 5), 0), (2, 1, (33, 31, 1), 1), (2, 3, (65, 9, 1), 0),
]
BOXES = [  # dim, k, base grid, box, walls
    (2, 1, (6, 6, 1), ((2, 2, 0), (4, 4, 0)), 0),
    (2, 3, (33, 8, 1), ((1, 1, 0), (32, 7, 0)), 1),
    (3, 1, (8, 6, 5), ((1, 1, 1), (7, 5, 4)), 0),
    (3, 2, (5, 5, 5), ((1, 2, 1), (4, 4, 4)), 1),
    (3, 3, (6, 5, 5), ((1, 1, 1), (5, 4, 4)), 0),
]
MTILDE = 2.0


def rough(shape, dim, dx, seed):
    r = np.random.default_rng(seed)
    w = r.uniform(-1, 1, size=shape) * (1.3 * MTILDE * dx / 3.0 ** 0.5)
    w[:, dim + 1:] *= 0.3
    c = shape[2:]
    thin = np.where(r.uniform(size=c) < 0.33, 0.02, 1.0)
    rho = thin * (1.0 + 0.2 * r.uniform(-1, 1, size=c))
    vel = [0.3 * r.uniform(-1, 1, size=c) for _ in range(dim)]
    w[0, 0] = rho
    for a in range(dim):
        w[1 + a, 0] = rho * vel[a]
    w[dim + 1, 0] = thin * (1.0 + 0.2 * r.uniform(-1, 1, size=c)) / 0.4 + 0.5 * rho * sum(v * v for v in vel)
    return w


def _changed(a, b):
    """[nvar][cells]: variables whose weights differ."""
    return (a != b).reshape(a.shape[0], a.shape[1], -1).any(axis=1)


def _partly(x, what):
    assert x.any() and not x.all(), (what, int(x.sum()), x.size)


def _run(dg, o, wl, w, blocks, case):
    """The limiter alone, positivity alone and both, against the oracle."""
    import torch
    for slope, posit in ((1, 0), (0, 1), (1, 1)):
        over = dict(wl, limiter=slope, positivity=posit)
        ref, st = o(over).limit(w.copy())
        assert st == 0
        for name, a, b in blocks(ref, w):
            x = _changed(a, b)
            if slope and not posit:
                _partly(x, (case, name, "limited variables"))
            if posit and not slope:
                _partly(x.any(axis=0), (case, name, "scaled cells"))
        s = dg.Solver(over)
        d = torch.from_numpy(np.ascontiguousarray(w)).cuda()
        s.limit(d)
        check_state(o(over), d.cpu().numpy(), ref, f"{case} slope {slope} positivity {posit}")
        assert s.status() == 0


@pytest.mark.parametrize("dim,k,n,walls", GRIDS)
def test_grids(dim, k, n, walls):
    import paper_1506_06140_amd as dg
    print("rough limit", dim, k, n, walls, flush=True)
    dx = 1.0 / 16
    wl = workloads.workload("kh3d" if dim == 3 else "density_wave", dim=dim, k=k, n=n, length=tuple(m * dx for m in n),
                            bc=(walls,) * dim + (0,) * (3 - dim), mtilde=MTILDE, rk="rk3")
    w = rough(oracle.Oracle(wl).shape, dim, dx, 3)
    _run(dg, oracle.Oracle, wl, w, lambda a, b: [("grid", a, b)], f"{n}")


@pytest.mark.parametrize("dim,k,n,box,walls", BOXES)
def test_boxes(dim, k, n, box, walls):
    import paper_1506_06140_amd as dg
    print("rough limit box", dim, k, n, box, walls, flush=True)
    dx = 1.0 / 8
    wl = workloads.workload("blast_amr", dim=dim, k=k, n=n, length=tuple(m * dx for m in n), refine_lo=box[0],
                            refine_hi=box[1], bc=(walls,) * dim + (0,) * (3 - dim), mtilde=MTILDE)
    o = oracle.AmrOracle(wl)
    w = o.initial_state()
    for i, b in enumerate(o.blocks(w)):  # views into w
        b[:] = rough(b.shape, dim, dx / (1 + i), 5 + i)

    def blocks(a, b):
        (ca, fa), (cb, fb) = o.blocks(a), o.blocks(b)
        return [("coarse", ca[:, :, ~o.hole], cb[:, :, ~o.hole]), ("fine", fa, fb)]

    _run(dg, oracle.AmrOracle, wl, w, blocks, f"{n} {box}")
