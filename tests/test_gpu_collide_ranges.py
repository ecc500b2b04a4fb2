"""Collision detection where its workgroups' ranges and their tables of entered
cells have edges: few markers, ranges that end inside a wavefront, far more
cells than the table holds, and cells contested by bodies of other workgroups.
Bit for bit the oracle."""
import numpy as np
import pytest

from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 65, 2049, 70001, 524289])
def test_ranges_and_entered_cells(orc, n):
    import torch
    from paper_1805_01113_amd import mls, workloads as W
    mls.load()
    gs = W.GridSpec([W.uniform_faces(48), W.uniform_faces(40), W.tanh_faces(33, 1.0, 1.5)], [True, True, False])
    r = np.random.default_rng(n)
    x, y, z = [r.uniform(0.0, 0.999, n).astype(np.float32) for _ in range(3)]
    # 1 + the cell's x index, and markers of other bodies in some cells
    body = (1 + np.floor(x.astype(np.float64) * 48)).astype(np.int32)
    other = r.random(n) < 0.02
    body[other] = r.integers(60, 70, int(other.sum()))
    ctx = mls.Context(gs.faces, gs.periodic)
    coll = torch.zeros(ctx.cell_shape(), dtype=torch.int32, device="cuda")
    flags = torch.empty(n, dtype=torch.uint8, device="cuda")
    pos = [to_dev(a) for a in (x, y, z)]
    ref = orc.collide(orc.Grid(gs.faces, gs.periodic), x, y, z, body)
    for _ in range(3):
        ctx.collide(*pos, torch.from_numpy(body).cuda(), coll, flags)
        ctx.sync()
        np.testing.assert_array_equal(coll.cpu().numpy(), ref["coll"])
        np.testing.assert_array_equal(flags.cpu().numpy(), ref["flag"])
        ctx.collide_clear(*pos, coll)
        ctx.sync()
        assert int(torch.count_nonzero(coll)) == 0
