"""Values at which the multigrid's operator has a zero to divide by or to raise
to a power: against the oracle, as everywhere 1e-12 of the largest value."""
import numpy as np
import pytest

import paper_2012_07322_amd as gmu
from oracle import mg
from test_gpu_mg import CART, CYL, D, N, PER, ROB, SPH, dev, host, prob

pytestmark = pytest.mark.gpu

# one level of the one-workgroup tail, 2D levels in place and out of place, 3D
# levels in place and out of place, one dimension, curvilinear, lines
GRIDS = {
    "1d": (1, CART, (64,), [[D, N]], {}),
    "2d_tail": (2, CART, (32, 24), [[D, N], [PER, PER]], {}),
    "2d_large": (2, CART, (256, 136), [[D, N], [D, D]], {}),
    "3d_tail": (3, CART, (16, 8, 12), [[D, N], [PER, PER], [D, D]], {}),
    "3d_in_place": (3, CART, (48, 40, 36), [[D, N], [PER, PER], [D, D]], {}),
    "3d_large": (3, CART, (160, 164, 162), [[D, N], [PER, PER], [D, D]], {}),
    "sph2d": (2, SPH, (32, 16), [[D, D], [N, N]], {}),
    "sph2d_line": (2, SPH, (32, 16), [[D, D], [N, N]], dict(smoother=gmu.MG_LINE)),
}


def grid(name, **kw):
    nd, coord, n, bc, opt = GRIDS[name]
    lo, hi = ((0.5, 0.3, 0.0), (2.5, 2.8, 1.0)) if coord == SPH else ((-1.0, -0.7, -0.4), (1.0, 0.9, 0.8))
    return prob(nd, coord, n, lo[:nd], hi[:nd], bc, levels=2, coarse=4, **opt, **kw)


def close(p, g, o):
    g, o = mg.interior(p, host(g)), mg.interior(p, o)
    assert np.isfinite(o).all()
    assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max()


@pytest.mark.parametrize("power", [0, 1])
@pytest.mark.parametrize("power2", [1, 2, 5])
@pytest.mark.parametrize("name", list(GRIDS))
def test_positive_power_of_zero(name, power, power2):
    """a (u + c)^p + a2 (u + c)^q at u + c = 0 with q > 0: from u = 0, c = 0."""
    p = grid(name, power=power, power2=power2, offset=0.0)
    rng = np.random.default_rng(23)
    shp = mg.shape(p)
    f, a, a2 = rng.uniform(-1, 1, shp), rng.uniform(0, 0.1, shp), rng.uniform(0.1, 1, shp)
    a = a if power else None
    M = gmu.Multigrid(p)
    fd, ad, a2d = dev(f), None if a is None else dev(a), dev(a2)
    o = np.zeros(shp)
    u = dev(o)
    assert M.residual_norm(u, fd, ad, a2d) == np.abs(mg.interior(p, f)).max()  # L(0) = 0
    (mg.line_smooth if p.get("smoother") else mg.smooth)(p, o, f, a, sweeps=2, a2=a2)
    close(p, M.smooth(u, fd, ad, sweeps=2, a2=a2d), o)
    o = np.zeros(shp)
    u = dev(o)
    opt = dict(tol=0.0, max_cycles=1, fmg=False)
    h = mg.solve(p, o, f, a, a2=a2, **opt)
    assert h[1] < h[0]  # the cycle contracts
    M.solve(u, fd, ad, a2=a2d, **opt)
    close(p, u, o)


def origin(nd, n, coord=CART, **kw):
    """A grid whose first cell's centre is the origin, with Robin faces on the
    lower sides: there the ghost's factor r_in / r_ghost is 0.  (Cylindrical:
    a ghost below the first cell of the axis, whose factor is not.)"""
    h = 0.125
    lo = [-0.5 * h] * nd if coord == CART else [0.0, -0.5 * h][:nd]
    bc = [[ROB if coord == CART or a else N, D if a % 2 else ROB] for a in range(nd)]
    return prob(nd, coord, n, lo, [x + h * m for x, m in zip(lo, n)], bc, levels=2, coarse=4, **kw)


ORIGIN = {
    "1d": origin(1, (64,)),
    "2d_tail": origin(2, (32, 24)),
    "2d_large": origin(2, (256, 136), power=1, offset=1.0),
    "3d_tail": origin(3, (16, 8, 12), power=-1, offset=2.0),
    "3d_in_place": origin(3, (48, 40, 36)),
    "3d_large": origin(3, (100, 104, 106)),
    "3d_large_a": origin(3, (100, 104, 106), power=1, offset=1.0),
    "3d_large_general": origin(3, (160, 164, 162), power=-1, offset=2.0),
    "cyl2d": origin(2, (32, 24), CYL),
    "2d_line": origin(2, (32, 24), smoother=gmu.MG_LINE),
}


@pytest.mark.parametrize("name", list(ORIGIN))
def test_robin_face_of_a_cell_at_the_origin(name):
    p = ORIGIN[name]
    rng = np.random.default_rng(29)
    shp = mg.shape(p)
    u0, f = 0.2 * rng.uniform(-1, 1, shp), rng.uniform(-1, 1, shp)
    a = rng.uniform(0, 0.1, shp) if p.get("power") else None
    M = gmu.Multigrid(p)
    fd, ad = dev(f), None if a is None else dev(a)
    o = mg.fill_ghosts(p, u0.copy())
    np.testing.assert_allclose(host(M.fill_ghosts(dev(u0))), o, rtol=1e-15, atol=0)
    L = mg.interior(p, f) - mg.interior(p, mg.apply(p, o, a))
    assert abs(M.residual_norm(dev(u0), fd, ad) - np.abs(L).max()) <= 1e-12 * np.abs(L).max()
    o = u0.copy()
    (mg.line_smooth if p.get("smoother") else mg.smooth)(p, o, f, a, sweeps=3)
    close(p, M.smooth(dev(u0), fd, ad, sweeps=3), o)
    o, u = u0.copy(), dev(u0)
    opt = dict(tol=0.0, max_cycles=1, fmg=False)
    h = mg.solve(p, o, f, a, **opt)
    assert h[1] < h[0]  # the cycle contracts
    M.solve(u, fd, ad, **opt)
    close(p, u, o)


@pytest.mark.parametrize("power2", [0, -7, -2])
def test_operator_at_a_zero_of_a_negative_power(power2):
    """u + c = 0 and infinite u with p = -1: the operator's infinities and
    NaNs are a division's."""
    p = dict(grid("3d_tail", power=-1, power2=power2, offset=1.0))
    rng = np.random.default_rng(31)
    shp = mg.shape(p)
    u, a = rng.uniform(0, 1, shp), rng.uniform(0.1, 1, shp)
    a2 = rng.uniform(0.1, 1, shp) if power2 else None
    u[4, 4, 4] = u[2, 6, 9] = -1.0
    a[2, 6, 9] = 0.0
    u[8, 5, 5] = np.inf
    o = mg.interior(p, mg.apply(p, u, a, a2))
    g = mg.interior(p, host(gmu.Multigrid(p).apply(dev(u), dev(a), a2=None if a2 is None else dev(a2))))
    assert np.array_equal(np.isnan(g), np.isnan(o)) and np.array_equal(np.isposinf(g), np.isposinf(o))
    assert np.array_equal(np.isneginf(g), np.isneginf(o)) and np.isneginf(o).any()
    ok = np.isfinite(o)
    assert np.abs(g[ok] - o[ok]).max() <= 1e-12 * np.abs(o[ok]).max()


@pytest.mark.parametrize("vector", [False, True])
def test_very_many_sweeps(vector):
    """A coarsest level relaxed by any number of sweeps is one launch (here to
    convergence; as launches of their own the cycle would be two million)."""
    p = prob(2, CART, (4, 4), (0.0, 0.0), (1.0, 1.0), [[D, N], [D, D]], coarse=(1 << 20) + 1)
    rng = np.random.default_rng(37)
    shp = (3,) * vector + mg.shape(p)
    f, o = rng.uniform(-1, 1, shp), np.zeros(shp)
    opt = dict(tol=0.0, max_cycles=1, fmg=False)
    M, u = gmu.Multigrid(p), dev(o)
    few = dict(p, coarse=400)  # converged as well
    (mg.vsolve if vector else mg.solve)(few, o, f, **opt)
    (M.vsolve if vector else M.solve)(u, dev(f), **opt)
    close(p, u, o)
