"""GPU: collision detection where the markers that lie next to each other in the
arrays are not of one body: a contact workload shuffled (the same cells and
flags as in order), and crowded cells that every body visits (about as fast as
the same markers spread over the grid, since a cell that is settled needs no
more atomics; with one per marker on 40 cells it is four times slower)."""
import pytest

from paper_1805_01113_amd import workloads as W
from parity import say

pytestmark = pytest.mark.gpu


def _collide(ctx, x, y, z, body):
    import torch
    coll = torch.zeros(ctx.cell_shape(), dtype=torch.int32, device="cuda")
    flags = torch.empty(x.numel(), dtype=torch.uint8, device="cuda")
    ctx.collide(x, y, z, body, coll, flags)
    return coll, flags


@pytest.mark.parametrize("n", [1, 64, 4097, 300001])
def test_shuffled_markers(n):
    import torch
    from paper_1805_01113_amd import mls
    g = torch.Generator("cuda").manual_seed(n)
    ctx = mls.Context([W.uniform_faces(48)] * 3, [True] * 3)
    body = torch.arange(n, device="cuda", dtype=torch.int32) // 500
    at = torch.rand((int(body[-1]) + 1, 3), generator=g, device="cuda")
    p = at[body.long()] + 0.1 * torch.rand((n, 3), generator=g, device="cuda")
    x, y, z = [p[:, d].contiguous() for d in range(3)]
    coll, flags = _collide(ctx, x, y, z, body)
    q = torch.randperm(n, device="cuda")
    coll2, flags2 = _collide(ctx, x[q].contiguous(), y[q].contiguous(), z[q].contiguous(), body[q].contiguous())
    ctx.sync()
    assert torch.equal(coll, coll2) and torch.equal(flags[q], flags2)
    assert n < 300000 or (coll == -1).any()


@pytest.mark.parametrize("bodies", [2, 1000])
def test_crowded_cells(bodies):
    import torch
    from paper_1805_01113_amd import mls
    n, m = 2000000, 64
    g = torch.Generator("cuda").manual_seed(bodies)
    ctx = mls.Context([W.uniform_faces(m)] * 3, [True] * 3)
    body = torch.randint(0, bodies, (n,), generator=g, device="cuda").to(torch.int32)
    cells = torch.randint(0, m, (40, 3), generator=g, device="cuda")
    inside = 0.1 + 0.8 * torch.rand((n, 3), generator=g, device="cuda")
    crowd = (cells[torch.randint(0, 40, (n,), generator=g, device="cuda")] + inside) / m
    spread = (torch.randint(0, m, (n, 3), generator=g, device="cuda") + inside) / m
    ms = []
    for p in (crowd, spread):
        x, y, z = [p[:, d].contiguous() for d in range(3)]
        best = 1e30
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            coll = torch.zeros(ctx.cell_shape(), dtype=torch.int32, device="cuda")
            flags = torch.empty(n, dtype=torch.uint8, device="cuda")
            a.record()
            ctx.collide(x, y, z, body, coll, flags)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
        k = (p * m).long()
        flat = (k[:, 2] * m + k[:, 1]) * m + k[:, 0]
        lo = torch.full((m ** 3,), 1 << 30, dtype=torch.int32, device="cuda").scatter_reduce_(0, flat, body, "amin")
        hi = torch.full((m ** 3,), -1, dtype=torch.int32, device="cuda").scatter_reduce_(0, flat, body, "amax")
        want = torch.where(hi < 0, 0, torch.where(lo == hi, lo + 1, -1)).reshape(m, m, m)
        assert torch.equal(coll, want.to(torch.int32))
        assert torch.equal(flags, (want.reshape(-1)[flat] == -1).to(torch.uint8))
    say("%d bodies: 40 cells %.3f ms, all cells %.3f ms" % (bodies, *ms))
    assert ms[0] < 2.5 * ms[1]
    ctx.sync()
