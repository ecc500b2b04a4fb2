"""The compact exact step on both sides of the size up to which its spreading goes
through the staging buffer, with every solve in FP64 and with a mixture (those
rows are finished by a second kernel), against the step with full rows: U, F,
the forcing, the routes and the FP64 rows' phi, bit for bit."""
import numpy as np
import pytest

from parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stretched", [False, True])
@pytest.mark.parametrize("n", [63, 4201, 4202, 9000])
@pytest.mark.parametrize("tau", [0.0, 11.0])
def test_compact_fp64_rows(n, tau, stretched):
    import torch
    from paper_1805_01113_amd import mls, workloads as W
    mls.load()
    # 18^3 tiles of 8 nodes: the boxes of 4201 fit the staging buffer
    faces = [W.uniform_faces(144), W.uniform_faces(144), W.tanh_faces(144, 1.0, 1.2) if stretched else W.uniform_faces(144)]
    r = np.random.default_rng(n)
    pos = [to_dev(r.uniform(0.03, 0.97, n).astype(np.float32)) for _ in range(3)]
    area = to_dev(r.uniform(0.2, 1.0, n).astype(np.float32) / 144 ** 2)
    ctx = mls.Context(faces, [True, True, not stretched], kappa_tau=tau)
    g = torch.Generator(device="cuda").manual_seed(5)
    grid = W.GridSpec(faces, [True, True, not stretched])
    fields = [torch.randn(grid.shape(c), generator=g, device="cuda") for c in range(3)]
    got = []
    for compact in (False, True):
        forcing = [torch.zeros(grid.shape(c), device="cuda") for c in range(3)]
        bufs = mls.StepBuffers(ctx, *pos, area, fields, forcing, route=True)
        bufs.phi.fill_(0)
        ctx.stats_reset()
        mls.step(ctx, bufs, method=mls.MLS_EXACT, dt=0.5, jitter=0.0, seed=0, compact=compact)
        ctx.sync()
        solves = ctx.stats()["fp64_solves"]
        order = mls.step_order(ctx, n).to(torch.int64)
        phi = torch.as_tensor(mls.unpack_phi(bufs.phi.cpu().numpy(), n))       # [3, n, 27] by row
        route = torch.as_tensor(mls.unpack_route(bufs.route.cpu().numpy(), n))    # [3, n] by row
        inv = torch.empty(n, dtype=torch.int64)
        inv[order.cpu()] = torch.arange(n)
        got.append((bufs.U.clone(), bufs.F.clone(), forcing, solves, phi[:, inv], route[:, inv]))
    full, comp = got
    assert full[3] == comp[3] and (tau > 0 or full[3] == 3 * n)
    if tau > 0 and n > 1000:
        assert 0 < full[3] < 3 * n
    assert torch.equal(full[0], comp[0]) and torch.equal(full[1], comp[1])
    assert all(torch.equal(a, b) for a, b in zip(full[2], comp[2]))
    assert torch.equal(full[5], comp[5])
    routed = full[5] == 1
    assert int(routed.sum()) == full[3]
    assert torch.equal(full[4][routed], comp[4][routed])
    assert not comp[4][~routed].any()
