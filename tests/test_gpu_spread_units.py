"""Spreading with every way of handing out its work: few workgroups (whole tiles,
claimed), many (tiles cut into components), 128 to 256 threads, compact and full
rows.  The fixed-point sums do not depend on any of it, so the step's forcing is
the same bit for bit; the standalone spreading, whose boxes keep the layers that
no support of the build reaches, agrees to the rounding of c_l F_l (1e-6
normwise: two FP32 roundings of each contribution)."""
import numpy as np
import pytest

from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stretched", [False, True])
def test_forcing_does_not_depend_on_the_hand_out(stretched):
    import torch
    from paper_1805_01113_amd import mls, workloads as W
    mls.load()
    m, n = 184, 60007
    faces = [W.uniform_faces(m), W.uniform_faces(m), W.tanh_faces(m, 1.0, 1.2) if stretched else W.uniform_faces(m)]
    gs = W.GridSpec(faces, [True, True, not stretched])
    r = np.random.default_rng(8)
    lo, hi = (0.03, 0.97) if stretched else (0.0, 1.0)
    pos = [to_dev(r.uniform(0.0, 1.0, n).astype(np.float32)) for _ in range(2)]
    pos.append(to_dev(r.uniform(lo, hi, n).astype(np.float32)))
    area = to_dev(r.uniform(0.2, 1.0, n).astype(np.float32) / m ** 2)
    ctx = mls.Context(faces, gs.periodic)
    g = torch.Generator(device="cuda").manual_seed(4)
    fields = [torch.randn(gs.shape(c), generator=g, device="cuda") for c in range(3)]
    first = None
    for compact in (True, False):
        for threads, per_cu in ((192, 8), (128, 1), (256, 1), (192, 32)):
            ctx.tune_set(spread_threads=threads, spread_blocks_per_cu=per_cu)
            forcing = [torch.zeros(gs.shape(c), device="cuda") for c in range(3)]
            bufs = mls.StepBuffers(ctx, *pos, area, fields, forcing)
            mls.step(ctx, bufs, method=mls.MLS_EXACT, dt=1.0, jitter=0.0, seed=0, compact=compact)
            ctx.sync()
            if first is None:
                first = forcing
                assert all(float(f.abs().max()) > 0 for f in first)
            assert all(torch.equal(a, b) for a, b in zip(first, forcing)), (compact, threads, per_cu)
    home, phi, _ = ctx.build(*pos, method=mls.MLS_EXACT)
    alone = [torch.zeros(gs.shape(c), device="cuda") for c in range(3)]
    ctx.spread(home, phi, area, bufs.F, alone)
    ctx.sync()
    for a, b in zip(first, alone):
        assert float((a - b).abs().max()) <= 1e-6 * float(a.abs().max())
