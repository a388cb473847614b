"""GPU: states past the sizes at which addressing or launching changes.

From 4 GB on (32-bit byte offsets) the 2D and 3D stages run on the kernels with
64-bit indices, the quadtree's and the adjoint's on their 64-bit forms.  A
small periodic grid repeated until its state is just above 4 GB has, in every
copy, the small grid's result: each element's copy that is furthest from the
oracle's value is held to the same bounds as the small grid's (the RHS to
1e-12 of fac(|V| + |S|), stages to 1e-12), the adjoint to 1e-12 of the small
grid's largest value (about 200 rounded terms, 2e-14)."""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_rhs_modes, check_state_modes

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


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _state(shape, dim, seed):
    """Means around (1, 0.4, -0.3, 0.2; p = 1) and modes of a few per cent."""
    r = np.random.default_rng(seed)
    w = 0.02 * r.uniform(-1, 1, size=shape)
    c = shape[2:]
    rho = 1.0 + 0.2 * r.uniform(-1, 1, size=c)
    vel = [b + 0.3 * r.uniform(-1, 1, size=c) for b in (0.4, -0.3, 0.2)[:dim]]
    w[0, 0] = rho
    for a in range(dim):
        w[1 + a, 0] = rho * vel[a]
    w[dim + 1, 0] = (1.0 + 0.2 * r.uniform(-1, 1, size=c)) / 0.4 + 0.5 * rho * sum(v * v for v in vel)
    return w


def _tiled(s, small, tiles):
    """The state of s that repeats small [nvar][N][nz][ny][nx] tiles (x, y, z) times."""
    import torch
    nv, N, nz, ny, nx = small.shape
    tx, ty, tz = tiles
    w = s.empty()
    w.view(nv, N, tz, nz, ty, ny, tx, nx).copy_(
        _dev(small).view(nv, N, 1, nz, 1, ny, 1, nx).expand(nv, N, tz, nz, ty, ny, tx, nx))
    assert w.numel() * 8 >= 2 ** 32
    torch.cuda.synchronize()
    return w


def _worst(got, ref, tiles):
    """Per element of the small grid the copy in got that is furthest from ref."""
    nv, N, nz, ny, nx = ref.shape
    tx, ty, tz = tiles
    g = got.view(nv, N, tz, nz, ty, ny, tx, nx)
    lo, hi = g.amin(dim=(2, 4, 6)).cpu().numpy(), g.amax(dim=(2, 4, 6)).cpu().numpy()
    assert not np.isnan(lo).any()
    return np.where(np.abs(lo - ref) > np.abs(hi - ref), lo, hi)


GRIDS = [  # dim, k, small grid, copies along each axis: 4.30 to 4.39 GB
    (2, 3, (50, 37, 1), (74, 100, 1)),
    (2, 4, (31, 33, 1), (100, 88, 1)),
    (3, 1, (20, 15, 12), (15, 20, 25)),
    (3, 2, (17, 13, 13), (13, 17, 17)),
    (3, 3, (16, 11, 11), (11, 16, 16)),
]


@pytest.mark.parametrize("dim,k,n,tiles", GRIDS)
def test_stage_above_4_gb(dim, k, n, tiles):
    import torch
    import paper_1506_06140_amd as dg
    print("above 4 GB", dim, k, flush=True)
    _room(24)
    name = "kh3d" if dim == 3 else "density_wave"
    over = dict(dim=dim, k=k, limiter=0, positivity=0, rk="rk3")
    o = oracle.Oracle(workloads.workload(name, n=n, length=tuple(m / 64 for m in n), **over))
    big = tuple(m * t for m, t in zip(n, tiles))
    s = dg.Solver(workloads.workload(name, n=big, length=tuple(m / 64 for m in big), **over))
    nz = n[2] if dim == 3 else 1
    shape = (dim + 2, s.N, nz, n[1], n[0])
    w, u = _state(shape, dim, 1), _state(shape, dim, 2)
    wd = _tiled(s, w, tiles)
    out = s.rhs(wd)
    V, S, A = (np.asarray(x).reshape(shape) for x in o.terms_cells(w.reshape(o.shape), with_abs=True))
    check_rhs_modes(_worst(out, V - S, tiles), V, S, A, f"{big} rhs")
    ref = np.asarray(o.rk3_stage(2, 1e-3, u.reshape(o.shape), w.reshape(o.shape))).reshape(shape)
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    s.rk_stage(2, dt, _tiled(s, u, tiles), wd, out)
    check_state_modes(_worst(out, ref, tiles), ref, f"{big} stage 2")
    assert s.status() == 0


@pytest.mark.parametrize("k,n,tiles", [(1, (50, 37, 1), (135, 181, 1)), (2, (50, 37, 1), (95, 128, 1)), (3, (50, 37, 1), (74, 100, 1))])
def test_adjoint_above_4_gb(k, n, tiles):
    import torch
    import paper_1506_06140_amd as dg
    print("adjoint above 4 GB", k, flush=True)
    _room(40)
    over = dict(dim=2, k=k, limiter=0, positivity=0, rk="rk3")
    small = dg.Solver(workloads.workload("density_wave", n=n, length=tuple(m / 64 for m in n), **over))
    big = tuple(m * t for m, t in zip(n, tiles))
    s = dg.Solver(workloads.workload("density_wave", n=big, length=tuple(m / 64 for m in big), **over))
    shape = (4, s.N, 1, n[1], n[0])
    r = np.random.default_rng(3)
    w, lam, acc = _state(shape, 2, 1), r.normal(size=shape), r.normal(size=shape)
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    flat = lambda a: _dev(a).view(small.shape)  # noqa: E731
    mu = small.adjoint_rhs(flat(w), flat(lam)).cpu().numpy().reshape(shape)
    wd, ld = _tiled(s, w, tiles), _tiled(s, lam, tiles)
    out = s.adjoint_rhs(wd, ld)
    assert np.abs(_worst(out, mu, tiles) - mu).max() <= 1e-12 * np.abs(mu).max()
    ref, aref = small.empty(), flat(acc)
    small.adjoint_rk_stage(2, dt, flat(w), flat(lam), aref.clone(), ref, aref)
    ad = _tiled(s, acc, tiles)
    s.adjoint_rk_stage(2, dt, wd, ld, ad, out, ad)
    for got, want in ((out, ref), (ad, aref)):
        x = want.cpu().numpy().reshape(shape)
        assert np.abs(_worst(got, x, tiles) - x).max() <= 1e-12 * np.abs(x).max()
    assert s.status() == 0


def test_adjoint_above_2_to_the_29_cells():
    """Planes of 4 GB and more: 64-bit lane addresses (k = 1; three states of 52 GB)."""
    import torch
    import paper_1506_06140_amd as dg
    print("adjoint above 2^29 cells", flush=True)
    _room(170)
    n, tiles = (50, 37, 1), (464, 626, 1)
    over = dict(dim=2, k=1, limiter=0, positivity=0, rk="rk3")
    small = dg.Solver(workloads.workload("density_wave", n=n, length=tuple(m / 64 for m in n), **over))
    big = tuple(m * t for m, t in zip(n, tiles))
    s = dg.Solver(workloads.workload("density_wave", n=big, length=tuple(m / 64 for m in big), **over))
    assert s.ncell >= 2 ** 29
    shape = (4, s.N, 1, n[1], n[0])
    w, lam = _state(shape, 2, 1), np.random.default_rng(3).normal(size=shape)
    mu = small.adjoint_rhs(_dev(w).view(small.shape), _dev(lam).view(small.shape)).cpu().numpy().reshape(shape)
    wd, ld = _tiled(s, w, tiles), _tiled(s, lam, tiles)
    out = s.adjoint_rhs(wd, ld)
    assert np.abs(_worst(out, mu, tiles) - mu).max() <= 1e-12 * np.abs(mu).max()
    assert s.status() == 0
    del wd, ld, out, s
    torch.cuda.empty_cache()


@pytest.mark.parametrize("k,n,flux", [(1, (14, 12), 0), (2, (14, 12), 1), (3, (14, 12), 0)])
def test_tree_stage_above_4_gb(k, n, flux):
    import torch
    import paper_1506_06140_amd as dg
    print("quadtree above 4 GB", k, flush=True)
    _room(24)
    leaves = np.asarray(workloads.random_tree(n, 2, 0.4, 11, periodic=(True, True)), dtype=np.int32)
    L, N = len(leaves), (k + 1) * (k + 2) // 2
    copies = -(-2 ** 32 // (8 * 4 * N * L))
    tx = int(copies ** 0.5) + 1
    ty = -(-copies // tx)
    over = dict(dim=2, k=k, limiter=0, positivity=0, rk="rk3", flux=flux)
    o = oracle.TreeOracle(workloads.workload("kh2d", n=(*n, 1), length=(n[0] / 64, n[1] / 64, 1.0), **over), leaves)
    at = np.stack(np.meshgrid(np.arange(ty), np.arange(tx), indexing="ij"), axis=-1).reshape(-1, 1, 2).astype(np.int32)
    every = np.repeat(leaves[None], tx * ty, axis=0)
    every[:, :, 1] += (at[:, :, 1] * n[0]) << leaves[:, 0]
    every[:, :, 2] += (at[:, :, 0] * n[1]) << leaves[:, 0]
    big = (n[0] * tx, n[1] * ty)
    s = dg.TreeSolver(workloads.workload("kh2d", n=(*big, 1), length=(big[0] / 64, big[1] / 64, 1.0), **over),
                      every.reshape(-1, 3))
    assert s.size * 8 >= 2 ** 32
    w, u = _state((4, N, L), 2, 1), _state((4, N, L), 2, 2)

    def tiled(a):
        return _dev(a)[:, :, None].expand(4, N, tx * ty, L).contiguous().view(s.shape)

    def worst(got, ref):
        g = got.view(4, N, tx * ty, L)
        lo, hi = g.amin(dim=2).cpu().numpy(), g.amax(dim=2).cpu().numpy()
        assert not np.isnan(lo).any()
        return np.where(np.abs(lo - ref) > np.abs(hi - ref), lo, hi)

    wd = tiled(w)
    out = s.rhs(wd)
    V, S, A = (np.asarray(x).reshape(4, N, L) for x in o.terms(w))
    check_rhs_modes(worst(out, V - S), V, S, A, f"{s.nleaf} leaves rhs")
    ref = np.asarray(o.rk3_stage(2, 1e-3, u, w)).reshape(4, N, L)
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    s.rk_stage(2, dt, tiled(u), wd, out)
    check_state_modes(worst(out, ref), ref, f"{s.nleaf} leaves stage 2")
    assert s.status() == 0


@pytest.mark.parametrize("k,n,lo,hi", [(2, (150, 140, 132), (30, 30, 30), (131, 129, 131)),
                                       (3, (112, 112, 112), (16, 16, 16), (96, 96, 97))])
def test_box_stage_above_4_gb(k, n, lo, hi):
    """The box has no copies to compare: the MFMA kernel (above 4 GB) against
    the vector kernels, whose contractions are in another order: to 1e-12 of
    the largest value of each variable (about 500 rounded terms, 1e-13)."""
    import torch
    import paper_1506_06140_amd as dg
    print("box above 4 GB", k, flush=True)
    _room(32)
    wl = workloads.workload("blast_amr", dim=3, k=k, n=n, refine_lo=lo, refine_hi=hi, limiter=0, positivity=0,
                            length=tuple(m / 64 for m in n))
    s, v = dg.Solver(wl), dg.Solver(dict(wl, path3d=dg.DG_PATH3D_VALU))
    w = s.empty()
    assert w.numel() * 8 >= 2 ** 32
    gen = torch.Generator(device="cuda").manual_seed(5)
    per = 5 * s.N
    blocks = lambda x: (x[:per * s.ncoarse].view(5, s.N, -1), x[per * s.ncoarse:].view(5, s.N, -1))  # noqa: E731
    for b in blocks(w):
        b.uniform_(-0.02, 0.02, generator=gen)
        b[0, 0] += 1.0
        for a, m in ((1, 0.4), (2, -0.3), (3, 0.2)):
            b[a, 0] += m
        b[4, 0] += 2.7
    got, ref = s.rhs(w), v.rhs(w)
    for g, r in zip(blocks(got), blocks(ref)):
        for i in range(5):
            scale = float(r[i].abs().max())
            assert scale > 0.0 and float((g[i] - r[i]).abs().max()) <= 1e-12 * scale
    assert s.status() == 0 and v.status() == 0
