"""The face ghosts that the recovery of a step writes equal a ghost fill of the
primitives it leaves, bit for bit, for every boundary rule and the faces where
the recovery leaves them to the ghost kernel."""
import math

import numpy as np
import pytest
import torch

import paper_2012_07322_amd as gmu
import workloads as W
from test_gpu_batch import make_batch
from test_gpu_parity import dev, host, smooth_random_state

pytestmark = pytest.mark.gpu

PER, OUT, REF, AXIS, CEN, NONE = range(6)
PI = math.pi
CASES = {
    "sph1d_centre": W.grid(1, W.SPH, [9], [0.0, 0.3, 0], [2.0, PI - 0.3, 2 * PI], [[CEN, OUT]]),
    "sph2d_centre_axis": W.grid(2, W.SPH, [11, 6], [0.0, 0.0, 0], [2.0, PI, 2 * PI], [[CEN, OUT], [AXIS, AXIS]]),
    "sph2d_equator": W.grid(2, W.SPH, [8, 5], [0.0, 0.0, 0], [2.0, PI / 2, 2 * PI], [[REF, OUT], [AXIS, REF]], ng=3),
    "sph3d_centre_axis": W.grid(3, W.SPH, [7, 6, 8], [0.0, 0.0, 0.0], [2.0, PI, 2 * PI],
                                [[CEN, OUT], [AXIS, AXIS], [PER, PER]], ng=3),
    "cyl2d_axis": W.grid(2, W.CYL, [6, 7], [0.0, -1.0, 0], [2.0, 1.0, 2 * PI], [[AXIS, OUT], [REF, OUT]]),
    "cyl3d_axis": W.grid(3, W.CYL, [5, 4, 6], [0.0, -1.0, 0.0], [2.0, 1.0, 2 * PI], [[AXIS, OUT], [OUT, OUT], [PER, PER]]),
    "cart3d_axis_in_z": W.grid(3, W.CART, [5, 4, 6], [0.3, 0.2, 0.1], [1.0, 1.1, 1.3], [[REF, OUT], [PER, PER], [AXIS, OUT]]),
    "cart3d_centre_in_y": W.grid(3, W.CART, [5, 4, 6], [0.3, 0.2, 0.1], [1.0, 1.1, 1.3], [[REF, OUT], [CEN, OUT], [PER, PER]]),
    "cart2d_none": W.grid(2, W.CART, [5, 4], [0.3, 0.2, 0.1], [1.0, 1.1, 1.3], [[OUT, OUT], [NONE, REF]]),
}


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("case", list(CASES))
def test_ghosts_after_a_step(case, batch):
    p = CASES[case]
    pr, met = smooth_random_state(p, beta_amp=0.0)
    g = gmu.Grid(p)
    if batch:
        B, views, _ = make_batch([(p, pr, met)], [0])
        B.step(1e-3, use_graph=False)
        prd = views[0][1].clone()
    else:
        prd, metd = dev(pr), dev(met)
        g.fill_ghosts(prd)
        qn = g.prim2con(prd, metd)
        t = torch.zeros(1, dtype=torch.float64, device="cuda")
        g.step(qn, torch.zeros_like(qn), prd, metd, 1e-3, 1e30, t, torch.zeros_like(t))
    filled = prd.clone()
    g.fill_ghosts(filled)
    assert np.isfinite(host(prd)).all()
    assert np.array_equal(host(prd), host(filled))
