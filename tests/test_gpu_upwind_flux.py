"""GPU: outside the star region the HLLC mass flux is the upwind momentum
itself.  Where the momentum is one value m everywhere and the flow supersonic
along every axis, all faces' mass fluxes are then the same number however the
density varies, and the mean density's tendency, a sum of +-that number (equal
along each axis, so every partial sum is 0 or the number), is exactly zero: the
cells' edge is a power of two, so scaling by 2/dx rounds nothing.  Formed as
rho (m / rho) the flux would be off by roundings of m."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

CASES = [(2, 1, (64, 5, 1)), (2, 2, (33, 17, 1)), (2, 3, (63, 4, 1)), (2, 4, (17, 9, 1)),
         (3, 1, (62, 5, 7)), (3, 2, (26, 26, 25)), (3, 3, (64, 3, 4))]


def supersonic(shape, dim, sign, seed):
    """Momentum components sign * 4, densities in (1, 2), pressures near 0.1: |u| > 2, c < 0.4."""
    r = np.random.default_rng(seed)
    w = np.zeros(shape)
    c = shape[2:]
    rho = 1.0 + r.uniform(size=c)
    w[0, 0] = rho
    w[1:1 + dim, 0] = 4.0 * sign
    w[dim + 1, 0] = 0.1 * (1.0 + 0.2 * r.uniform(size=c)) / 0.4 + 0.5 * dim * 16.0 / rho
    return w


def _grid(dim, k, n, flux):
    return workloads.workload("kh3d" if dim == 3 else "density_wave", dim=dim, k=k, n=n, flux=flux, limiter=0,
                              positivity=0, rk="rk3", length=tuple(m / 64 for m in n))


@pytest.mark.parametrize("flux", [0, 1])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("dim,k,n", CASES)
def test_mass_flux_is_the_momentum(dim, k, n, sign, flux):
    import torch
    import paper_1506_06140_amd as dg
    print("upwind flux", dim, k, n, sign, flux, flush=True)
    s = dg.Solver(_grid(dim, k, n, flux))
    w = supersonic(s.shape, dim, sign, 3)
    L = s.rhs(torch.from_numpy(w).cuda()).cpu().numpy()
    assert np.abs(L[0, 0]).max() == 0.0
    assert np.abs(L[dim + 1, 0]).max() > 0.0 and s.status() == 0


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_mass_flux_is_the_momentum_tree(k, sign):
    import torch
    import paper_1506_06140_amd as dg
    print("upwind flux tree", k, sign, flush=True)
    n = (13, 5)
    wl = workloads.workload("kh2d", k=k, n=(*n, 1), length=(n[0] / 8, n[1] / 8, 1.0), limiter=0, positivity=0, rk="rk3")
    s = dg.TreeSolver(wl, workloads.random_tree(n, 0, 0.4, 11, periodic=(True, True)))
    w = supersonic(s.shape, 2, sign, 5)
    L = s.rhs(torch.from_numpy(w).cuda()).cpu().numpy()
    assert np.abs(L[0, 0]).max() == 0.0
    assert np.abs(L[3, 0]).max() > 0.0 and s.status() == 0


@pytest.mark.parametrize("flux", [0, 1])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_adjoint_of_the_mass_flux(k, sign, flux):
    """The reverse sweep of the same faces: the mass flux depends on the upwind
    cell's momentum alone, with slope one.  A cotangent on the mean density's
    tendency only then reaches no density and no energy (exactly zero), and a
    cell's momentum along an axis by 2 fac times the cotangent's difference to
    the downwind neighbour (k + 1 rounded terms: 8 eps)."""
    import torch
    import paper_1506_06140_amd as dg
    print("upwind adjoint", k, sign, flux, flush=True)
    n = (33, 17, 1)
    s = dg.Solver(_grid(2, k, n, flux))
    w = supersonic(s.shape, 2, sign, 3)
    lam = np.zeros(s.shape)
    lam[0, 0] = np.random.default_rng(9).integers(-8, 8, size=s.shape[2:])
    mu = s.adjoint_rhs(torch.from_numpy(w).cuda(), torch.from_numpy(lam).cuda()).cpu().numpy()
    assert np.abs(mu[0]).max() == 0.0 and np.abs(mu[3]).max() == 0.0
    fac = 2.0 * 64 / 4
    for a in range(2):
        d = np.roll(lam[0, 0], -1, axis=2 - a) - lam[0, 0] if sign > 0 else lam[0, 0] - np.roll(lam[0, 0], 1, axis=2 - a)
        assert np.abs(mu[1 + a, 0] - 2.0 * fac * d).max() <= 8 * 2.0 ** -52 * 2.0 * fac * 16
    assert s.status() == 0
