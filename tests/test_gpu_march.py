"""The marched stage of large Cartesian 3D grids at the sizes where it can go
wrong (remainders of its columns of 31x7 and 15x15 cells, last chunks of one
plane), against the oracle and against the tile kernel that a block of a
batch takes.

Tile and marched stage evaluate the same terms in the same order and differ
where the compiler fuses a product into a sum, so two steps agree to the
1e-12 of the variable's (or its vector's) scale that the limited stages are
compared with: a few hundred roundings of 1.1e-16 per cell and step on states
whose recovery is well conditioned (rho, p of order 1, v < 0.5)."""
import numpy as np
import pytest
import torch

import test_gpu_pp
import workloads as W
from test_gpu_batch import alone, make_batch
from test_gpu_parity import rhs_check, smooth_kij, smooth_random_state

pytestmark = pytest.mark.gpu

# cells, options; the comment names the column and the planes of a workgroup
GRIDS = [
    ((62, 49, 129), {}),                                # 31x7, 4: exact columns, a last chunk of one plane
    ((94, 36, 113), dict(riemann=1)),                   # 31x7, 5: one cell over in x and y
    ((75, 45, 113), {}),                                # 15x15, 4: exact columns, a last chunk of one plane
    ((76, 91, 61), dict(riemann=1)),                    # one cell over in x and y
    ((63, 45, 129), dict(rk=2)),                        # 15x15, 4
    ((62, 57, 73), dict(recon=1, ng=3)),                # MP5, 15x15, 4
    ((61, 46, 97), dict(recon=1, riemann=1, ng=3)),     # one cell over
    ((62, 57, 73), dict(recon=2, ng=3)),                # PPM
]
IDS = ["x".join(map(str, n)) + "".join(f"-{k}{v}" for k, v in o.items()) for n, o in GRIDS]


def _grid(n, opt, beta):
    p = W.grid(3, W.CART, list(n), [-1.0, -0.8, -1.2], [1.0, 0.9, 1.1], [[1, 1], [0, 0], [2, 2]], **opt)
    pr, met = smooth_random_state(p, beta_amp=beta)
    if beta == 0.0:  # flat in the half x < 0, so that planes of both kinds meet
        x1 = W.centres(p)[0]
        met[0] = np.where(x1 < 0.0, 1.0, met[0])
        met[1] = np.where(x1 < 0.0, 1.0, met[1])
    return p, pr, met


def _cells(n, seed=5):
    """Random cells and every combination of cells about the columns' edges."""
    rng = np.random.default_rng(seed)
    out = [np.stack([rng.integers(0, m, 800) for m in n], axis=1)]
    at = [sorted({c for e in es for c in (e - 1, e, m - 1 - e) if 0 <= c < m})
          for m, es in zip(n, ([0, 15, 30, 31, 62], [0, 7, 15, 35], [0, 1, 4, 5]))]
    out.append(np.array([(i, j, k) for i in at[0] for j in at[1] for k in at[2]]))
    return np.concatenate(out).astype(np.int32)


@pytest.mark.parametrize("beta", [0.05, 0.0])
@pytest.mark.parametrize("n,opt", GRIDS, ids=IDS)
def test_rhs_parity(n, opt, beta):
    p, pr, met = _grid(n, opt, beta)
    rhs_check(p, pr, met, cells=_cells(n))


def test_rhs_parity_with_supplied_kij():
    p, pr, met = _grid(*GRIDS[0], 0.05)
    rhs_check(p, pr, met, cells=_cells(GRIDS[0][0]), kij=smooth_kij(p))


@pytest.mark.parametrize("beta", [0.05, 0.0])
@pytest.mark.parametrize("n,opt", GRIDS, ids=IDS)
def test_steps_agree_with_a_batch_block(n, opt, beta):
    p, pr, met = _grid(n, opt, beta)
    B, views, _ = make_batch([(p, pr, met)], [0])
    for _ in range(2):
        B.step(0.3, use_graph=False)
    torch.cuda.synchronize()
    qa, pa, _ = alone(p, pr, met, 2, cfl=0.3)
    g = p["ng"]
    inner = (slice(None),) + (slice(g, -g),) * 3
    for a, b in ((qa, views[0][0]), (pa, views[0][1])):
        a, b = a[inner], b.cpu().numpy()[inner]
        for grp in ([0], [1, 2, 3], [4], [5, 6, 7]):  # vector components share their vector's scale
            assert np.abs(a[grp] - b[grp]).max() <= 1e-12 * np.abs(b[grp]).max(), grp


@pytest.mark.parametrize("axis,riemann", [(2, 0), (0, 1)])
def test_limited_stage_parity(monkeypatch, axis, riemann):
    """MP5 (the other reconstructions' limited stages stay on tiles)."""
    flow = test_gpu_pp._flow
    monkeypatch.setattr(test_gpu_pp, "_flow", lambda *a, **k: flow(*a, ng=3, recon=1, **k))
    test_gpu_pp.test_limited_stage_parity(W.CART, 3, axis, None, (62, 57, 73), riemann)


@pytest.mark.parametrize("n,opt", [
    ((17, 104, 88), dict(recon=2, ng=3)),               # columns of 9 and 8 cells
    ((32, 97, 101), dict(recon=1, riemann=1, ng=3)),    # 11, 11 and 10
    ((46, 226, 45), {}),                                # 12, 12, 11 and 11
    ((15, 210, 88), dict(recon=2, ng=3)),               # one column
], ids=["17", "32", "46", "15"])
def test_rhs_parity_of_columns_shared_out_along_x(n, opt):
    p, pr, met = _grid(n, opt, 0.05)
    cells = [(i, j, k) for i in range(n[0]) for j in (0, 14, 15, n[1] - 1) for k in (0, 3, 4, n[2] - 1)]
    rhs_check(p, pr, met, cells=np.array(cells, dtype=np.int32))
