"""One multigrid cycle against the oracle at the level sizes where the GPU's
kernels change: levels at, just below and above the largest that the
one-workgroup tail of the hierarchy takes (4096 cells), odd and very flat
coarsest levels, one, two or many levels, one and three sweeps.

Both sides run the same sweeps on the same O(1) data in FP64 with another
operation order, and a cycle that reduces the residual contracts differences:
1e-12 of the largest |u|.
"""
import numpy as np
import pytest

import paper_2012_07322_amd as gmu
from oracle import mg
from test_gpu_mg import CART, CYL, D, N, PER, ROB, SPH, dev, host, prob

pytestmark = pytest.mark.gpu

BOX = ((-1.0, -0.7, -0.4), (1.0, 0.9, 0.8))


def cart(n, *bc, **kw):
    return prob(len(n), CART, n, BOX[0][:len(n)], BOX[1][:len(n)], bc, **kw)


SCALAR = {
    "2d_4096": cart((64, 64), [D, N], [PER, PER]),
    "2d_above_4096": cart((66, 64), [D, D], [N, D], coarse=3),
    "2d_flat": cart((512, 4), [D, ROB], [N, ROB]),
    "1d_4096": cart((4096,), [D, N], coarse=4),
    "3d_4096": cart((16, 16, 16), [ROB, ROB], [ROB, ROB], [ROB, ROB]),
    "3d_odd_coarsest": cart((12, 20, 28), [D, D], [N, D], [D, ROB]),
    "3d_one_level": cart((6, 5, 3), [D, D], [N, D], [D, D], levels=1, coarse=7),
    "3d_two_levels": cart((36, 20, 12), [D, D], [PER, PER], [D, N], levels=2, coarse=6, pre=1, post=3),
    "3d_32": cart((32, 48, 40), [PER, PER], [D, ROB], [N, D], pre=3, post=1),
    "2d_big": cart((160, 224), [D, ROB], [N, D]),
    "cyl3d": prob(3, CYL, (24, 32, 16), (0.0, -1, 0), (2.0, 1, 6.2), [[N, ROB], [ROB, D], [PER, PER]]),
    "sph2d": prob(2, SPH, (96, 32), (0.0, 0.0), (4.0, 1.5), [[N, ROB], [N, N]]),
}


@pytest.mark.parametrize("fmg", [True, False])
@pytest.mark.parametrize("terms", ["linear", "a_lin", "a_inv_a2"])
@pytest.mark.parametrize("name", list(SCALAR))
def test_one_cycle(name, terms, fmg):
    p = dict(SCALAR[name])
    p.update({"linear": dict(power=0), "a_lin": dict(power=1, offset=1.0),
              "a_inv_a2": dict(power=-1, offset=1.0, power2=-7)}[terms])
    rng = np.random.default_rng(7)
    shp = mg.shape(p)
    u, f = 0.2 * rng.uniform(-1, 1, shp), rng.uniform(-1, 1, shp)
    a = None if terms == "linear" else rng.uniform(0.1, 1, shp) * (1 if terms == "a_lin" else -1)
    a2 = -rng.uniform(0, 0.1, shp) if terms == "a_inv_a2" else None
    uo, opt = u.copy(), dict(tol=0.0, max_cycles=1, fmg=fmg)
    h = mg.solve(p, uo, f, a, a2=a2, **opt)
    if not h[1] < h[0]:
        pytest.skip("the oracle's own cycle diverges from this start: nothing contracts")
    ug = dev(u)
    gmu.Multigrid(p).solve(ug, dev(f), None if a is None else dev(a), a2=None if a2 is None else dev(a2), **opt)
    g, o = mg.interior(p, host(ug)), mg.interior(p, uo)
    assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max()


VECTOR = {
    "2d_1024": cart((32, 32), [D, N], [PER, PER]),
    "2d_above_1024": cart((34, 32), [D, D], [N, D], coarse=3),
    "1d": cart((1024,), [D, N], coarse=4),
    "3d_above_1024": cart((12, 12, 8), [N, N], [PER, PER], [D, D]),
    "3d_flat": cart((64, 4, 2), [D, N], [N, D], [N, N]),
    "3d_one_level": cart((6, 5, 3), [D, D], [N, D], [D, D], levels=1, coarse=7),
    "3d_odd_coarsest": cart((12, 20, 28), [D, N], [N, D], [D, D], pre=3, post=1),
    "3d_wide": cart((72, 36, 40), [PER, PER], [D, N], [N, D], pre=1, post=1),
    "2d_big": cart((160, 224), [D, N], [N, D]),
}


@pytest.mark.parametrize("fmg", [True, False])
@pytest.mark.parametrize("name", list(VECTOR))
def test_one_vector_cycle(name, fmg):
    p = VECTOR[name]
    rng = np.random.default_rng(11)
    X, f = rng.uniform(-1, 1, (3,) + mg.shape(p)), rng.uniform(-1, 1, (3,) + mg.shape(p))
    Xo, opt = X.copy(), dict(tol=0.0, max_cycles=1, fmg=fmg)
    h = mg.vsolve(p, Xo, f, **opt)
    if not h[1] < h[0]:
        pytest.skip("the oracle's own cycle diverges from this start: nothing contracts")
    Xg = dev(X)
    gmu.Multigrid(p).vsolve(Xg, dev(f), **opt)
    g = host(Xg)
    for c in range(3):
        a, b = mg.interior(p, g[c]), mg.interior(p, Xo[c])
        assert np.abs(a - b).max() <= 1e-12 * np.abs(Xo).max(), c


@pytest.mark.parametrize("coord", [SPH, CYL])
@pytest.mark.parametrize("n", [(2, 65), (64, 64), (65, 3), (682, 2), (683, 4)], ids=lambda n: "x".join(map(str, n)))
def test_line_sweeps_where_the_kernels_change(coord, n):
    """Lines of one and two wavefronts, the longest whose two components are
    solved together and the first that are not, along both axes of
    axisymmetric grids.  Two sweeps against the oracle's elimination: the
    line systems' condition number is about n^2 in units of eps, each
    sweep's two axes and the second component on top of the first: 4 n^2 eps,
    at least 1e-12."""
    lo, hi, bc = ((0.0, 0.0), (4.0, np.pi / 2), [[N, D], [N, N]]) if coord == SPH else (
        (0.0, -1.0), (4.0, 1.5), [[N, D], [N, D]])
    p = prob(2, coord, n, lo, hi, bc, smoother=gmu.MG_LINE)
    rng = np.random.default_rng(13)
    X, f = rng.uniform(-1, 1, (3,) + mg.shape(p)), rng.uniform(-1, 1, (3,) + mg.shape(p))
    Xg = dev(X)
    gmu.Multigrid(p).vsmooth(Xg, dev(f), sweeps=2)
    Xo = mg.vline_smooth(p, X.copy(), f, sweeps=2)
    tol = max(1e-12, 4.0 * max(n) ** 2 * np.finfo(float).eps)
    g = host(Xg)
    for c in range(3):
        assert np.abs(mg.interior(p, g[c]) - mg.interior(p, Xo[c])).max() <= tol * np.abs(Xo).max(), c
