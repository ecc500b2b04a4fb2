"""GPU: the network's passes in a caller's graph follow the parameters that are
loaded, whether the load comes before the capture, after it or between replays.

The expected values are those of a context that loads the same parameters and
runs eagerly: the same kernels on the same operands, so the same bits.
"""
import numpy as np
import pytest

from paper_1805_01113_amd import workloads as W

pytestmark = pytest.mark.gpu


def _net(seed):
    r = np.random.default_rng(seed)
    p = r.normal(0.0, 0.15, 20891).astype(np.float32)
    norm = np.concatenate([r.normal(0.0, 0.3, 6), r.uniform(0.5, 2.0, 6)]).astype(np.float32)
    return p, norm


def _ctx():
    from paper_1805_01113_amd import mls
    return mls.Context([W.uniform_faces(16)] * 3, [True] * 3)


def _batch(m):
    import torch
    g = torch.Generator("cuda").manual_seed(m)
    feat = torch.rand((m, 6), generator=g, device="cuda") - 0.5
    feat[:, 3:] = 1.0
    return feat, torch.rand((m, 27), generator=g, device="cuda")


def _eager(net, feat, target):
    ctx = _ctx()
    ctx.mlp_load(*net)
    loss, grad = ctx.mlp_grad(feat, target)
    out = [ctx.mlp_forward(feat), loss, grad]
    ctx.sync()
    return out


@pytest.mark.parametrize("m", [1, 33, 1000])
def test_captured_passes_follow_a_load(m):
    import torch
    feat, target = _batch(m)
    nets = [_net(s) for s in range(3)]
    want = [_eager(n, feat, target) for n in nets]
    ctx = _ctx()
    ctx.mlp_load(*nets[0])
    ctx.mlp_grad(feat, target)          # scratch of the batch
    ctx.mlp_forward(feat)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = [ctx.mlp_forward(feat)]
        out += ctx.mlp_grad(feat, target)
    for k in (0, 1, 2, 0):
        ctx.mlp_load(*nets[k])
        for _ in range(2):
            for t in out:
                t.fill_(-7.0)
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(out, want[k]):
                assert torch.equal(a, b)
    ctx.sync()


@pytest.mark.parametrize("m", [33])
def test_eager_pass_between_capture_and_replay(m):
    import torch
    feat, target = _batch(m)
    nets = [_net(s) for s in range(2)]
    want = [_eager(n, feat, target) for n in nets]
    ctx = _ctx()
    ctx.mlp_load(*nets[0])
    ctx.mlp_grad(feat, target)
    torch.cuda.synchronize()
    ctx.mlp_load(*nets[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = [ctx.mlp_forward(feat)]
        out += ctx.mlp_grad(feat, target)
    first = [ctx.mlp_forward(feat), *ctx.mlp_grad(feat, target)]
    torch.cuda.synchronize()
    for a, b in zip(first, want[1]):
        assert torch.equal(a, b)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want[1]):
            assert torch.equal(a, b)
    # a training step moves the parameters: the graph and an eager pass agree
    ctx.mlp_train_step(feat, target, lr=1e-3)
    now = [ctx.mlp_forward(feat), *ctx.mlp_grad(feat, target)]
    graph.replay()
    torch.cuda.synchronize()
    for a, b, c in zip(out, now, want[1]):
        assert torch.equal(a, b) and not torch.equal(a, c)
    ctx.sync()
