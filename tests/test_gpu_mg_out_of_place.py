"""The red-black sweeps that large levels run out of place (3D Cartesian levels
from 2^20 cells, others and those with a general term from 2^22; 2D levels
above 4096 cells) against the oracle's sweeps and cycle: every boundary rule on
every axis, each kind of term and coordinates, tiles of 32 x 16 cells and
chunks of planes with remainders, one and two sweeps per launch.

Both sides run the same sweeps on the same O(1) data in FP64 with another
operation order, and a sweep contracts differences: 1e-12 of the largest |u|.
"""
import math

import numpy as np
import pytest

import paper_2012_07322_amd as gmu
from oracle import mg
from test_gpu_mg import CART, CYL, D, N, PER, ROB, SPH, dev, host, prob

pytestmark = pytest.mark.gpu

LO, HI = (-0.9, -0.6, 0.0), (1.0, 0.8, 1.1)


def cart(n, *bc, **kw):
    return prob(len(n), CART, n, LO[:len(n)], HI[:len(n)], bc, **{"levels": 1, **kw})


LINEAR, GENERAL = dict(power=1, offset=1.0), dict(power=-1, offset=2.0, power2=-7)

SWEEPS = {
    # 2^20 cells: one resident round of workgroups, last chunks of 2 to 10 planes
    "robin_xy_periodic_z": cart((100, 102, 104), [ROB, ROB], [N, ROB], [PER, PER]),
    "robin_x_periodic_yz_a": cart((96, 104, 112), [D, ROB], [PER, PER], [PER, PER], **LINEAR),
    "robin_yz_periodic_x": cart((352, 58, 54), [PER, PER], [ROB, N], [D, ROB]),
    "robin_all_a": cart((101, 103, 105), [ROB, ROB], [ROB, ROB], [ROB, ROB], **LINEAR),
    "odd": cart((101, 103, 105), [D, N], [N, D], [D, N]),
    "odd_a": cart((101, 103, 105), [N, D], [D, D], [N, N], **LINEAR),
    "periodic_z": cart((130, 90, 92), [D, N], [N, D], [PER, PER]),
    "periodic": cart((66, 130, 126), [PER, PER], [PER, PER], [PER, PER], **LINEAR),
    # 2^22 cells: a general term or curvilinear weights; two rounds of workgroups
    "linear_large": cart((162, 161, 163), [D, N], [N, D], [D, N], **LINEAR),
    "general": cart((162, 161, 163), [D, N], [N, D], [D, N], **GENERAL),
    "general_robin_xy_periodic_z": cart((160, 162, 164), [ROB, D], [N, ROB], [PER, PER], **GENERAL),
    "general_flat": cart((64, 66, 1000), [PER, PER], [ROB, ROB], [ROB, D], **GENERAL),
    "cyl": prob(3, CYL, (160, 162, 164), (0.0, -1.0, 0.0), (2.0, 1.0, 2 * math.pi), [[N, ROB], [ROB, D], [PER, PER]],
                levels=1, **LINEAR),
    "sph": prob(3, SPH, (160, 162, 164), (0.5, 0.3, 0.0), (2.5, math.pi - 0.3, 2 * math.pi),
                [[D, ROB], [N, D], [PER, PER]], levels=1, **GENERAL),
    # 2D
    "2d_periodic": cart((258, 130), [PER, PER], [PER, PER], **LINEAR),
    "2d_robin_periodic": cart((130, 258), [ROB, D], [PER, PER]),
    "2d_odd_general": cart((257, 129), [ROB, N], [D, ROB], **GENERAL),
}


def fields(p, seed):
    rng = np.random.default_rng(seed)
    shp = mg.shape(p)
    u, f = rng.uniform(-1, 1, shp), rng.uniform(-1, 1, shp)
    a = rng.uniform(0, 0.1, shp) if p.get("power") else None
    a2 = rng.uniform(0, 0.1, shp) if p.get("power2") else None
    return u, f, a, a2


def opt(a):
    return None if a is None else dev(a)


@pytest.mark.parametrize("name", list(SWEEPS))
def test_sweeps(name):
    p = SWEEPS[name]
    u, f, a, a2 = fields(p, 17)
    M = gmu.Multigrid(p)
    fd, ad, a2d = dev(f), opt(a), opt(a2)
    # two sweeps are two launches of one, three a launch of two and one of one, four two of two
    for sweeps in (2, 3, 4):
        ug = dev(u)
        M.smooth(ug, fd, ad, sweeps=sweeps, a2=a2d)
        uo = mg.smooth(p, u.copy(), f, a, sweeps=sweeps, a2=a2)
        g, o = mg.interior(p, host(ug)), mg.interior(p, uo)
        assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max(), sweeps


CYCLES = {
    "robin_xy_periodic_z": cart((96, 104, 112), [ROB, ROB], [N, ROB], [PER, PER], levels=4, coarse=8),
    "robin_x_periodic_yz_a": cart((96, 104, 112), [D, ROB], [PER, PER], [PER, PER], levels=3, coarse=8, pre=1, post=3,
                                  **LINEAR),
    "2d_periodic": cart((100, 72), [PER, PER], [PER, PER], levels=2, coarse=8, **LINEAR),
    "2d_robin_periodic": cart((72, 100), [ROB, D], [PER, PER], levels=2, coarse=8, pre=3),
}


@pytest.mark.parametrize("name", list(CYCLES))
def test_one_cycle(name):
    p = CYCLES[name]
    u, f, a, a2 = fields(p, 19)
    uo = 0.2 * u
    ug = dev(uo)
    o = dict(tol=0.0, max_cycles=1, fmg=False)
    h = mg.solve(p, uo, f, a, a2=a2, **o)
    assert h[1] < h[0]  # the cycle contracts
    gmu.Multigrid(p).solve(ug, dev(f), opt(a), a2=opt(a2), **o)
    g, o = mg.interior(p, host(ug)), mg.interior(p, uo)
    assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max()
