"""Multigrid with little device memory left: the second fields of the
out-of-place sweeps are optional, so that a refused allocation of one relaxes
its level in place and the calls succeed.  In place and out of place are the
same sweeps in another operation order: 1e-12 of the largest value."""
import gc

import pytest
import torch

import paper_2012_07322_amd as gmu
from test_gpu_mg import CART, D, N, prob

pytestmark = pytest.mark.gpu


def box(n):
    return prob(3, CART, (n, n, n), (-1, -1, -1), (1, 1, 1), [[D, N], [D, D], [N, D]])


def fill(leave):
    """Take the device's free memory but about `leave` bytes (at most that
    and 32 MB; what the driver reports as free follows an allocation roughly)."""
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hog = []
    for _ in range(12):
        more = torch.cuda.mem_get_info()[0] - leave
        if more < 32 << 20:
            break
        try:
            hog.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:  # fragmented: in smaller pieces
            hog.append(torch.empty(more // 4, dtype=torch.uint8, device="cuda"))
    if not leave // 2 < torch.cuda.mem_get_info()[0] < leave + (32 << 20):
        hog.clear()
        torch.cuda.empty_cache()
        pytest.skip("the device's free memory could not be brought to the size of the test")
    return hog


def fields(M, vector):
    gen = torch.Generator(device="cuda").manual_seed(5)
    e = M.empty(vector=vector)
    return tuple(torch.rand(e.shape, generator=gen, device="cuda", dtype=torch.float64) - 0.5 for _ in range(2))


def run(M, vector, u, f):
    (M.vsolve if vector else M.solve)(u, f, tol=0.0, max_cycles=2, fmg=False)
    return u


def check(M, vector, u, f, want, leave):
    hog = fill(leave) if leave else None
    try:
        run(M, vector, u, f)
        err = M.residual_norm(u, f) if not vector else 0.0  # (reports an error left behind, too)
    finally:
        del hog
        torch.cuda.empty_cache()
    assert err == err
    assert float((u - want).abs().max()) <= 1e-12 * float(want.abs().max())


@pytest.mark.parametrize("vector,n", [(False, 512), (True, 256)])
def test_solve_without_memory_for_the_finest_second_field(vector, n):
    """512^3: the second field takes 1.09 GB; 256^3 vector: the coarse levels'
    arrays 0.3 GB, the finest second field 0.41 GB; 0.6 GB are left."""
    M = gmu.Multigrid(box(n))
    u, f = fields(M, vector)
    want = run(M, vector, u.clone(), f)
    M.close()
    M = gmu.Multigrid(box(n))
    check(M, vector, u, f, want, 600 << 20)
    M.close()


def test_create_without_memory_for_the_coarse_second_fields():
    """512^3: with half of what the second fields of the 256^3 and 128^3 levels
    take left beside the arrays that a hierarchy cannot do without."""
    M = gmu.Multigrid(box(512))
    u, f = fields(M, False)
    want = run(M, False, u.clone(), f)
    size = [torch.Size(M.shape(l)).numel() * 8 for l in range(M.levels)]
    second = sum(s for l, s in enumerate(size[:-1]) if 2 ** (3 * (l + 1)) >= 1 << 20)
    M.close()
    hog = fill(size[-1] + 5 * sum(size[:-1]) + second // 2)
    try:
        M = gmu.Multigrid(box(512))
    finally:
        del hog
        torch.cuda.empty_cache()
    check(M, False, u, f, want, 0)
    M.close()
