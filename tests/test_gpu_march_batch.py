"""Large Cartesian 3D grids march their stage along z alone, in a batch and in
the server: the same bits on each path, on columns of both shapes with one cell
over, exact or one short along x and y, and last chunks of every length; the
right-hand side against the oracle.  The route of each grid (its column, and by
the count of items the planes of a chunk) is asserted."""
import numpy as np
import pytest
import torch

import paper_2012_07322_amd as gmu
import workloads as W
from test_gpu_batch import alone, blast_like_blocks, make_batch
from test_gpu_parity import rhs_check, smooth_random_state
from test_gpu_serving import alone as served_alone
from test_gpu_serving import collect

pytestmark = pytest.mark.gpu

COLUMNS = [(31, 7), (15, 15), (15, 15), (15, 15)]  # of the library's marched stages, after its 14 tile shapes
TILES = 14

# cells, options, column, planes per chunk
GRIDS = [
    ((187, 22, 85), {}, 0, 5),                              # one cell over in x and y
    ((310, 29, 37), dict(riemann=1, rk=2), 0, 4),           # exact, one over; a last chunk of one plane
    ((216, 13, 109), {}, 0, 4),                             # one short in x and y
    ((46, 226, 45), dict(riemann=1), 1, 6),                 # one over in x and y
    ((136, 15, 169), dict(rk=2), 1, 4),                     # one over, exact; one plane
    ((104, 29, 109), {}, 1, 4),                             # one short
    ((91, 46, 53), dict(recon=1, ng=3), 2, 4),              # MP5: one over in x and y; one plane
    ((44, 29, 161), dict(recon=1, riemann=1, ng=3), 2, 4),  # one short
    ((91, 46, 53), dict(recon=2, riemann=1, ng=3), 3, 4),   # PPM
    ((180, 21, 53), dict(recon=2, rk=2, ng=3), 3, 4),       # exact, six over
]
IDS = ["x".join(map(str, n)) + "".join(f"-{k}{v}" for k, v in o.items()) for n, o, _, _ in GRIDS]


def make(n, opt, beta=0.05):
    p = W.grid(3, W.CART, list(n), [-1.0, -0.8, -1.2], [1.0, 0.9, 1.1], [[1, 1], [0, 0], [2, 2]], **opt)
    pr, met = smooth_random_state(p, beta_amp=beta)
    if beta == 0.0:  # flat in the half x < 0, so that planes of both kinds meet
        x1 = W.centres(p)[0]
        met[0] = np.where(x1 < 0.0, 1.0, met[0])
        met[1] = np.where(x1 < 0.0, 1.0, met[1])
    return p, pr, met


def items(n, col, zlen):
    tx, ty = COLUMNS[col]
    return -(-n[0] // tx) * -(-n[1] // ty) * -(-n[2] // zlen)


def same(p, views, q, prim):
    a, b = W.interior(p, views[0].cpu().numpy()), W.interior(p, q)
    differ = int((a != b).sum()), int((views[1].cpu().numpy() != prim).sum())
    assert differ == (0, 0)


@pytest.mark.parametrize("beta", [0.05, 0.0])
@pytest.mark.parametrize("n,opt,col,zlen", GRIDS, ids=IDS)
def test_block_equals_alone(n, opt, col, zlen, beta):
    p, pr, met = make(n, opt, beta)
    B, views, _ = make_batch([(p, pr, met)], [0])
    it, var = B.info()
    assert var[0] == TILES + col and it[0] == items(n, col, zlen)
    for graph in (False, True):
        B.step(0.3, use_graph=graph)
    torch.cuda.synchronize()
    q, prim, t = alone(p, pr, met, 2, cfl=0.3)
    assert B.times()[0][0] == t
    same(p, views[0], q, prim)


@pytest.mark.parametrize("n,opt,col,zlen", GRIDS, ids=IDS)
def test_rhs_parity(n, opt, col, zlen):
    p, pr, met = make(n, opt)
    B, _, _ = make_batch([(p, pr, met)], [0])
    assert B.info()[1][0] == TILES + col  # the route that the grid alone takes too
    rng = np.random.default_rng(5)
    cells = [np.stack([rng.integers(0, m, 600) for m in n], axis=1)]
    tx, ty = COLUMNS[col]
    edges = [range(0, m + s, s) for m, s in zip(n, (tx, ty, zlen))]
    at = [sorted({c for e in es for c in (e - 1, e) if 0 <= c < m}) for m, es in zip(n, edges)]
    at = [a if len(a) < 8 else a[:4] + a[-4:] for a in at]
    cells.append(np.array([(i, j, k) for i in at[0] for j in at[1] for k in at[2]]))
    rhs_check(p, pr, met, cells=np.concatenate(cells).astype(np.int32))


@pytest.mark.parametrize("n,opt", [g[:2] for g in GRIDS if g[2] != 2],
                         ids=[i for i, g in zip(IDS, GRIDS) if g[2] != 2])
def test_limited_stage_on_tiles_agrees(n, opt):
    """With MC and PPM a limited stage stays on tiles where the unlimited one
    marches.  Where every theta is 1 both are the same terms in the same order:
    1e-12 of the variable's (or its vector's) scale."""
    p, pr, met = make(n, opt)
    dt = torch.full((1,), 1e-4, dtype=torch.float64, device="cuda")
    out = []
    for pp in (0, 1):
        g = gmu.Grid(dict(p, pp_limiter=pp))
        prd, metd = torch.from_numpy(pr.copy()).cuda(), torch.from_numpy(met).cuda()
        g.fill_ghosts(prd)
        qn = g.prim2con(prd, metd)
        qs, q = qn.clone(), torch.zeros_like(qn)
        g.rk_stage(1, dt, qn, qs, q, prd, prd, metd)
        torch.cuda.synchronize()
        out.append((W.interior(p, q.cpu().numpy()), W.interior(p, prd.cpu().numpy())))
    for a, b in zip(*out):
        for grp in ([0], [1, 2, 3], [4], [5, 6, 7]):
            assert np.abs(a[grp] - b[grp]).max() <= 1e-12 * np.abs(b[grp]).max(), grp


def test_marching_blocks_beside_tiles():
    """Marching blocks of every column shape and small blocks in one batch,
    groups that stop at different times, several steps per replay, blocks that
    come and go under one captured step; a pinned or tuned tile shape leaves a
    marching block as it is."""
    big = [make(n, {k: v for k, v in opt.items() if k != "rk"}) for n, opt, _, _ in GRIDS[::2]]
    blocks = big + blast_like_blocks()
    groups = list(range(len(blocks)))
    B, views, _ = make_batch(blocks, groups)
    for p, _, _ in big[:2]:
        B.set_tile(p, 16, 4, 3)
    B.autotune()
    var = B.info()[1]
    assert [v >= TILES for v in var[:len(blocks)]] == [True] * len(big) + [False] * 3
    B.set_group(1, 0.0, 1e30, max_steps=2)
    B.commit()
    steps = [4] * len(blocks)
    steps[1] = 2
    B.steps(0.3, 3)
    B.clear_block(0)  # the replayed step no longer holds it
    steps[0] = 3
    B.commit()
    B.steps(0.3, 1)
    torch.cuda.synchronize()
    t = B.times()[0]
    for k, (p, pr, met) in enumerate(blocks):
        q, prim, ta = alone(p, pr, met, steps[k], cfl=0.3)
        assert k == 0 or t[k] == ta, k
        same(p, views[k], q, prim)


def test_capacity_is_counted_in_tiles():
    """A batch refuses a marching block exactly where it refuses the block's
    tiles."""
    n, opt, _, _ = GRIDS[6]
    p, pr, met = make(n, opt)
    tiles = -(-n[0] // 8) * -(-n[1] // 5) * -(-n[2] // 5)
    a = [torch.from_numpy(pr.copy()).cuda() for _ in range(3)] + [torch.from_numpy(met).cuda()]
    for cap, ok in ((tiles - 1, False), (tiles, True)):
        B = gmu.Batch(1, 1, cap)
        B.set_block(0, p, *a, 0)
        if ok:
            B.commit()
        else:
            with pytest.raises(RuntimeError):
                B.commit()
        B.close()


def test_served_solve_equals_alone():
    """A large 3D solve among smaller ones, of both integrators."""
    probs = []
    spec = [(3, 72, 3, 5), (3, 14, 3, 6), (2, 272, 3, 4), (3, 80, 2, 5), (1, 300, 2, None)]
    for i, (kind, n, rk, ms) in enumerate(spec):
        p, pr, met, te, m0 = W.serving_problem({"kind": kind, "n": n, "seed": 60 + i, "arrival": 0.0}, "cuda")
        p["rk"] = rk
        probs.append((p, pr, met, te, m0 if ms is None else ms))
    for p, pr, met, _, _ in (probs[0], probs[3]):
        B, _, _ = make_batch([(p, pr.cpu().numpy(), met.cpu().numpy())], [0])
        assert B.info()[1][0] >= TILES
    S = gmu.Server(1 << 30, max_slots=8, cfl=0.4, steps_per_sync=2)
    outs = []
    for k, (p, pr, met, te, ms) in enumerate(probs):
        out = torch.empty_like(pr), torch.empty_like(pr)
        S.submit(p, pr, met, te, ms, q_out=out[0], prim_out=out[1], tag=k)
        outs.append(out)
    res = {r["tag"]: r for r in collect(S, len(probs))}
    S.close()
    for k, (p, pr, met, te, ms) in enumerate(probs):
        assert res[k]["status"] == 0 and res[k]["nfatal"] == 0, res[k]
        q, prim, t = served_alone(p, pr, met, te, ms)
        assert res[k]["t"] == t
        assert torch.equal(W.interior(p, q), W.interior(p, outs[k][0])) and torch.equal(prim, outs[k][1]), k
