"""GPU: gradients of fields that are NaN where a solver holds no values.  A pair
with a NaN in its support is NaN in value and gradient and is not solved again,
so a call on such fields takes about the time it takes on clean ones; a NaN just
outside the support, or across a periodic edge, changes nothing for it."""
import numpy as np
import pytest

from paper_1805_01113_amd import workloads as W
from parity import say

pytestmark = pytest.mark.gpu


def _best(call, reps=5):
    import torch
    best = 1e30
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("pressure", [False, True])
def test_all_nan(pressure):
    """Solved again in FP64 every pair takes ten times a clean call; three times allows for noise."""
    import torch
    from paper_1805_01113_amd import mls
    n = 500000
    g = W.GridSpec([W.uniform_faces(96)] * 3, [True] * 3)
    ctx = mls.Context(g.faces, g.periodic)
    p = torch.rand((3, n), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    p = p[:, torch.argsort((p * 96).long().mul(torch.tensor([[1], [96], [96 * 96]], device="cuda")).sum(0))]
    pos = [v.contiguous() for v in p]      # cell by cell, as the markers of a surface are near each other
    shapes = [g.shape(c) for c in range(3)] + [ctx.cell_shape()]
    clean = [torch.rand(s, device="cuda") for s in shapes]
    nan = [torch.full(s, float("nan"), device="cuda") for s in shapes]

    def call(f):
        return ctx.interp_grad(*pos, *f[:3], p=f[3] if pressure else None)

    out = call(nan)
    for t in out.values():
        assert t is None or torch.isnan(t).all()
    for t in call(clean).values():
        assert t is None or torch.isfinite(t).all()
    t_nan, t_clean = _best(lambda: call(nan)), _best(lambda: call(clean))
    say("all NaN %.3f ms, clean %.3f ms" % (t_nan, t_clean))
    assert t_nan < 3.0 * t_clean
    assert ctx.stats()["fp64_solves"] == 0
    ctx.sync()


@pytest.mark.parametrize("d", [0, 1, 2])
def test_nan_beside_the_support(d):
    """Homes in the first cells of a periodic axis: an infinite value at its last node is in the support, a NaN at
    node 2 or 3 may be just outside it."""
    import torch
    from paper_1805_01113_amd import mls
    m, n = 12, 4000
    g = W.GridSpec([W.uniform_faces(m)] * 3, [True] * 3)
    ctx = mls.Context(g.faces, g.periodic)
    r = np.random.default_rng(d)
    p = r.uniform(0.0, 1.0, (3, n)).astype(np.float32)
    p[d] = (r.uniform(-0.6, 2.0, n) / m).astype(np.float32)
    pos = [torch.from_numpy(v).cuda() for v in p]
    f = []
    for c in range(3):
        q = np.ascontiguousarray(r.uniform(1.0, 2.0, (m, m, m)).astype(np.float32))
        view = np.moveaxis(q, 2 - d, 0)
        view[-1] = np.inf
        view[2 + c % 2] = np.nan
        f.append(q)
    out = ctx.interp_grad(*pos, *[torch.from_numpy(q).cuda() for q in f])
    k = np.arange(27)
    for c in range(3):
        home, phi, _ = ctx.build_grad(*pos, c)
        h = home.cpu().numpy().view(np.uint32)[:n].astype(np.int64)
        ph = phi.permute(0, 2, 1).reshape(-1, 27)[:n].double().cpu().numpy()
        idx = [(h & 2047)[:, None] + k % 3 - 1, (h >> 11 & 2047)[:, None] + k // 3 % 3 - 1,
               (h >> 22)[:, None] + k // 9 - 1]
        q = f[c].astype(np.float64)[idx[2] % m, idx[1] % m, idx[0] % m]
        nan, inf = np.isnan(q).any(1), np.isinf(q).any(1)
        got = out["U"][c].double().cpu().numpy()
        grad = out["G"][3 * c:3 * c + 3].cpu().numpy()
        assert np.isnan(got[nan]).all() and np.isnan(grad[:, nan]).all()
        assert np.isfinite(got[~nan & ~inf]).all() and np.isfinite(grad[:, ~nan & ~inf]).all()
        only = inf & ~nan & (np.abs(ph) > 1e-6).all(1)
        with np.errstate(invalid="ignore"):
            want = (ph * q).sum(1)
        assert only.sum() > 100 and (nan.sum() > 100 or c == 1)     # (node 3 is out of reach)
        assert np.array_equal(np.isnan(got[only]), np.isnan(want[only]))
        sure = only & ~np.isnan(want)
        assert np.array_equal(got[sure], want[sure])
    ctx.sync()
