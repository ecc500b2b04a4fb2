"""GPU: cells and home nodes of markers within a few FP32 steps of faces and
cell centres, on axes that do not start at 0 (where the FP32 lookup's bound has
all its terms, or does not hold at all), in every direction: homes of the exact
build and cells of the collision detection against the oracle's, exactly.
"""
import numpy as np
import pytest

from paper_1805_01113_amd import workloads as W
from parity import to_dev

pytestmark = pytest.mark.gpu

AXES = {
    "uniform, origin -3.7": (W.uniform_faces(517, 2.2, -3.7), True),
    "uniform, origin 1000": (W.uniform_faces(300, 1.0, 1000.0), True),
    "uniform, origin 1e-3": (W.uniform_faces(64, 1.0, 1e-3), True),
    "uniform walls, origin 5.3": (W.uniform_faces(130, 0.7, 5.3), False),
    "stretched walls, origin -1.5": (W.tanh_faces(128, 3.0, 2.5) - 1.5, False),
    "stretched, periodic, origin 7": (W.tanh_faces(96, 2.0, 1.5) + 7.0, True),
}


def _near(r, f, periodic, lo, hi):
    """FP32 coordinates in [lo, hi): at random, and up to three steps from faces and centres (periodic: from their
    images too)."""
    at = np.concatenate([f, 0.5 * (f[:-1] + f[1:])])
    if periodic:
        at = np.concatenate([at, at - (f[-1] - f[0]), at + (f[-1] - f[0])])
    steps = [at.astype(np.float32)]
    for way in (-np.inf, np.inf):
        v = steps[0]
        for _ in range(3):
            v = np.nextafter(v, np.float32(way))
            steps.append(v)
    x = np.concatenate(steps + [r.uniform(lo, hi, 2000).astype(np.float32)])
    x = x[(x.astype(np.float64) >= lo) & (x.astype(np.float64) < hi)]
    return r.permutation(x)


@pytest.mark.parametrize("d", [0, 1, 2])
@pytest.mark.parametrize("name", AXES)
def test_cells_and_homes_near_faces(orc, name, d):
    import torch
    from paper_1805_01113_amd import mls
    f, periodic = AXES[name]
    r = np.random.default_rng(len(f) + d)
    other = W.uniform_faces(8)
    faces = [f if k == d else other for k in range(3)]
    per = [periodic if k == d else True for k in range(3)]
    ctx, og = mls.Context(faces, per), orc.Grid(faces, per)
    L = f[-1] - f[0]
    # homes: on a wall axis where the supports of faces and of centres fit
    lo, hi = (f[0] - 0.3 * L, f[-1] + 0.3 * L) if periodic else (f[1], f[-2])
    along = _near(r, f, periodic, lo, hi)
    n = len(along)
    pos = [along if k == d else r.uniform(0.0, 1.0, n).astype(np.float32) for k in range(3)]
    home, _, _ = ctx.build(*[to_dev(p) for p in pos], method=mls.MLS_EXACT)
    ctx.sync()
    h = mls.unpack_home(home.cpu().numpy().view(np.uint32), n)
    for c in range(3):
        assert np.array_equal(h[c], orc.build_exact(og, c, *pos)["home"]), (name, d, c)
    # the time step bins from the positions and locates them again
    grid = W.GridSpec(faces, per)
    fields = [torch.ones(grid.shape(c), device="cuda") for c in range(3)]
    bufs = mls.StepBuffers(ctx, *[to_dev(p) for p in pos], torch.full((n,), 1e-3, device="cuda"), fields,
                           [torch.zeros_like(v) for v in fields])
    mls.step(ctx, bufs, method=mls.MLS_EXACT)
    ctx.sync()                             # a home outside its tile's box would be reported
    order = mls.step_order(ctx, n).cpu().numpy().astype(np.int64)
    assert np.array_equal(mls.unpack_home(bufs.home.cpu().numpy().view(np.uint32), n), h[:, order])
    # cells: the whole axis; a body a marker, so that every cell shows who is in it
    along = _near(r, f, periodic, *((lo, hi) if periodic else (f[0], f[-1])))
    n = len(along)
    pos = [along if k == d else r.uniform(0.0, 1.0, n).astype(np.float32) for k in range(3)]
    body = np.arange(n, dtype=np.int32)
    coll = torch.zeros(ctx.cell_shape(), dtype=torch.int32, device="cuda")
    flags = torch.empty(n, dtype=torch.uint8, device="cuda")
    ctx.collide(*[to_dev(p) for p in pos], torch.from_numpy(body).cuda(), coll, flags)
    ctx.sync()
    ref = orc.collide(og, *pos, body)
    assert np.array_equal(coll.cpu().numpy(), ref["coll"]), (name, d)
    assert np.array_equal(flags.cpu().numpy(), ref["flag"])
