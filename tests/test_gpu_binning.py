"""GPU: the tile scan of the spreading over its three ways of finding a
chunk's offset (from the counts of the chunks before it, from their sums, from
their scanned sums), at the sizes where one gives way to the next, and the
spreading in two launches against one launch per colour.

A chunk is 2048 tiles; up to 8 chunks a block adds up counts, up to 4096 it
adds up sums.  A time step scans one bucket more than a stand-alone call, so
16384 tiles are 8 chunks for the one and 9 for the other.  The forcing is
compared with the oracle's and, for the largest tiling, with that of tiles of
eight cells on the same markers: the two round each of at most eight box sums
per node to FP32 (6e-8 each) over fixed-point sums of 2^-30 of four times a
tile's largest force, so they agree to 1e-6 of the largest value.
"""
import numpy as np
import pytest

from paper_1805_01113_amd import workloads as W
from parity import F_TOL, normwise, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _markers(n, count, seed):
    r = np.random.default_rng(seed)
    pos = r.random((3, count)) * (np.asarray(n) / n[0])[:, None]
    return pos.astype(np.float32), r.uniform(0.2, 1.0, count).astype(np.float32) / n[0] ** 2, \
        r.normal(size=(3, count)).astype(np.float32)


@pytest.mark.parametrize("n,tile", [((16, 16, 16), 4), ((128, 128, 64), 4), ((128, 128, 68), 4)])
def test_scan_of_few_and_many_chunks(torch_cuda, n, tile):
    from oracle import oracle as orc
    from paper_1805_01113_amd import mls
    torch = torch_cuda
    g = W.GridSpec([W.uniform_faces(n[d], n[d] / n[0]) for d in range(3)], [True] * 3)
    pos, area, force = _markers(n, 3001, 11)
    ctx = mls.Context(g.faces, g.periodic, spread_tile=tile)
    x, y, z, a = [torch.from_numpy(v).cuda() for v in (*pos, area)]
    home, phi, _ = ctx.build(x, y, z)
    f = [torch.zeros(g.shape(c), device="cuda") for c in range(3)]
    ctx.spread(home, phi, a, torch.from_numpy(force).cuda(), f)
    fields = [torch.rand(g.shape(c), device="cuda", generator=torch.Generator("cuda").manual_seed(c))
              for c in range(3)]
    fs = [torch.zeros(g.shape(c), device="cuda") for c in range(3)]
    bufs = mls.StepBuffers(ctx, x, y, z, a, fields, fs)
    mls.step(ctx, bufs)
    ctx.sync()
    og = orc.Grid(g.faces, g.periodic)
    for c in range(3):
        ref = orc.build_exact(og, c, *pos)
        fo, _ = orc.spread(og, c, ref["home"], ref["phi"], area, force[c])
        so, _ = orc.spread(og, c, ref["home"], ref["phi"], area, bufs.F[c].cpu().numpy())
        e, es = normwise(f[c].cpu().numpy(), fo), normwise(fs[c].cpu().numpy(), so)
        say("tiles %s comp %d: spread %.2e step %.2e" % (ctx.stats()["spread_tiles"], c, e, es))
        assert e <= F_TOL and es <= F_TOL


def test_scan_of_the_largest_tilings(torch_cuda):
    """8,388,608 tiles: 4096 chunks for a stand-alone call, 4097 for a step."""
    from paper_1805_01113_amd import mls
    torch = torch_cuda
    n = (1024, 1024, 512)
    g = W.GridSpec([W.uniform_faces(n[d], n[d] / n[0]) for d in range(3)], [True] * 3)
    pos, area, force = _markers(n, 20011, 12)
    x, y, z, a = [torch.from_numpy(v).cuda() for v in (*pos, area)]
    fields = [torch.rand(g.shape(c), device="cuda", generator=torch.Generator("cuda").manual_seed(c))
              for c in range(3)]
    out = []
    for tile in (8, 4):
        ctx = mls.Context(g.faces, g.periodic, spread_tile=tile)
        home, phi, _ = ctx.build(x, y, z)
        f = [torch.zeros(g.shape(c), device="cuda") for c in range(3)]
        ctx.spread(home, phi, a, torch.from_numpy(force).cuda(), f)
        bufs = mls.StepBuffers(ctx, x, y, z, a, fields, [torch.zeros_like(v) for v in f])
        mls.step(ctx, bufs)
        ctx.sync()
        assert ctx.stats()["spread_entries"] == pos.shape[1]
        out.append(f + bufs.forcing)
        ctx.close()
    for p, q in zip(*out):
        top = float(p.abs().max())
        assert top > 0.0 and float((p - q).abs().max()) <= 1e-6 * top


@pytest.mark.parametrize("n,wall,tile,count", [
    ((16, 24, 32), False, 8, 700),       # one whole axis, three tiles (odd), four tiles
    ((24, 24, 24), False, 12, 1),        # two tiles an axis: both neighbours are the same tile
    ((20, 35, 18), False, 5, 65),        # tiles of 5, 5 or 7, and 9 or 6 cells
    ((32, 40, 21), True, 8, 900),        # a last tile cut short by the wall
    ((48, 16, 64), True, 16, 4000),      # the largest boxes
    ((64, 64, 64), False, 4, 20000),     # many small, crowded tiles
])
def test_two_launches_equal_colour_launches(torch_cuda, n, wall, tile, count):
    """mls_spread takes two launches through its staging buffer where the boxes
    fit it, mls_spread_noalloc always one launch per colour: the forcing, added
    to fields that are not zero, is the same bit for bit."""
    from paper_1805_01113_amd import mls
    torch = torch_cuda
    g = W.GridSpec([W.uniform_faces(n[d], n[d] / n[0]) for d in range(3)], [True, True, not wall])
    pos, area, force = _markers(n, count, 13)
    if wall:
        lo, hi = 1.5 / n[0], (n[2] - 1.5) / n[0]
        pos[2] = np.clip(pos[2], np.float32(lo), np.float32(hi))
    ctx = mls.Context(g.faces, g.periodic, spread_tile=tile)
    x, y, z, a = [torch.from_numpy(v).cuda() for v in (*pos, area)]
    F = torch.from_numpy(force).cuda()
    home, phi, _ = ctx.build(x, y, z)
    start = [torch.randn(g.shape(c), device="cuda", generator=torch.Generator("cuda").manual_seed(c))
             for c in range(3)]
    one, two = [v.clone() for v in start], [v.clone() for v in start]
    ctx.spread_noalloc(home, phi, a, F, one)
    ctx.spread(home, phi, a, F, two)
    ctx.sync()
    for c in range(3):
        assert torch.equal(one[c], two[c])
        assert not torch.equal(one[c], start[c])
