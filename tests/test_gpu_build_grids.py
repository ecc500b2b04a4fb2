"""The builds where their grids change: the marker counts around one resident
round of workgroups (504 of full rows, 768 of compact rows and of the standalone
build, four wavefronts each, three wavefronts per 64 markers), where wavefronts
begin to stride.  Every marker must be built once by its own row: the step's rows,
by marker, against the standalone build, and the compact step's U and F against
the full step's, bit for bit (the same arithmetic from the same positions)."""
import numpy as np
import pytest

from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64 * 672, 64 * 672 + 1, 64 * 1024, 64 * 1024 + 1, 64 * 2048 + 63])
def test_every_marker_is_built(n):
    import torch
    from paper_1805_01113_amd import mls, workloads as W
    mls.load()
    gs = W.GridSpec([W.uniform_faces(96), W.uniform_faces(80), W.tanh_faces(64, 1.0, 1.4)], [True, True, False])
    r = np.random.default_rng(n)
    pos = [to_dev(r.uniform(0.03, 0.97, n).astype(np.float32)) for _ in range(3)]
    area = to_dev(r.uniform(0.2, 1.0, n).astype(np.float32) / 96 ** 2)
    ctx = mls.Context(gs.faces, gs.periodic)
    g = torch.Generator(device="cuda").manual_seed(3)
    fields = [torch.randn(gs.shape(c), generator=g, device="cuda") for c in range(3)]
    home, phi, _ = ctx.build(*pos, method=mls.MLS_EXACT)
    ctx.sync()
    want = (mls.unblock(home, n)[:, :, 0], mls.unpack_phi(phi, n))
    U = []
    for compact in (False, True):
        forcing = [torch.zeros(gs.shape(c), device="cuda") for c in range(3)]
        bufs = mls.StepBuffers(ctx, *pos, area, fields, forcing)
        bufs.U.fill_(float("nan"))
        bufs.F.fill_(float("nan"))
        mls.step(ctx, bufs, method=mls.MLS_EXACT, dt=1.0, jitter=0.0, seed=0, compact=compact)
        ctx.sync()
        order = mls.step_order(ctx, n).to(torch.int64)
        assert torch.equal(torch.sort(order)[0], torch.arange(n, device="cuda"))
        assert torch.equal(mls.unblock(bufs.home, n)[:, :, 0], want[0][:, order])
        if not compact:
            assert torch.equal(mls.unpack_phi(bufs.phi, n), want[1][:, order])
        U.append((bufs.U.clone(), bufs.F.clone()))
        assert torch.isfinite(bufs.U).all() and torch.isfinite(bufs.F).all()
    assert torch.equal(U[0][0], U[1][0]) and torch.equal(U[0][1], U[1][1])
