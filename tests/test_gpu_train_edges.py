"""GPU: the training kernels at the batch sizes where their cuts change -- 16
samples a workgroup, batches padded to 32, chunks of at least 128 samples and at
most 64 of them -- against the FP64 oracle on identical FP32 parameters.

Tolerances as for the whole network in 32-bit accumulation with split-BF16
products (2^-17 relative each): outputs 2e-4 and gradient blocks 1e-4 normwise.
"""
import numpy as np
import pytest

from parity import normwise, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net():
    import torch
    assert torch.cuda.is_available()
    from oracle import mlp as M
    from paper_1805_01113_amd import mls, workloads as W
    r = np.random.default_rng(21)
    p = M.init_params(4)
    p.b1, p.b2, p.b3 = r.normal(0, 0.3, 128), r.normal(0, 0.3, 128), r.normal(0, 0.05, 27)
    p.shift = np.array([0.0, 0.0, 0.0, 1.0, 1.0, 1.0])
    p.scale = np.array([3.4, 3.4, 3.4, 1.0, 1.0, 40.0])
    flat = p.flat().astype(np.float32)
    norm = np.concatenate([p.shift, p.scale]).astype(np.float32)
    q = M.Params.unflat(flat.astype(np.float64), norm[:6].astype(np.float64), norm[6:].astype(np.float64))
    ctx = mls.Context([W.uniform_faces(16)] * 3, [True] * 3)
    ctx.mlp_load(flat, norm)
    rows = 9000
    feat = np.ones((rows, 6), dtype=np.float32)
    feat[:, :3] = r.uniform(-0.5, 0.5, (rows, 3))
    feat[:, 5] = np.exp(r.normal(0, 0.02, rows))
    target = r.normal(0, 0.3, (rows, 27)).astype(np.float32)
    return M, ctx, q, feat, target, torch.from_numpy(feat).cuda(), torch.from_numpy(target).cuda()


@pytest.mark.parametrize("m", [1, 15, 16, 17, 31, 33, 127, 128, 129, 8192, 8193])
def test_gradient_at_batch_edges(net, m):
    M, ctx, q, feat, target, fd, td = net
    y = ctx.mlp_forward(fd[:m].contiguous())
    loss, grad = ctx.mlp_grad(fd[:m].contiguous(), td[:m].contiguous(), mu=1.0)
    ctx.sync()
    ref, _ = M.forward(q, feat[:m].astype(np.float64))
    L, G = M.loss_and_grad(q, feat[:m].astype(np.float64), target[:m].astype(np.float64), mu=1.0)
    ey, el = normwise(y.cpu().numpy(), ref), abs(float(loss.item()) - L) / abs(L)
    gg = grad.cpu().numpy()
    offs = np.cumsum([0, 768, 128, 16384, 128, 3456, 27])
    eg = [normwise(gg[a:b], G[a:b]) for a, b in zip(offs[:-1], offs[1:])]
    say("batch %d: outputs %.2e loss %.2e gradient blocks %s" % (m, ey, el, ["%.1e" % e for e in eg]))
    assert ey <= 2e-4 and el <= 1e-4 and max(eg) <= 1e-4
