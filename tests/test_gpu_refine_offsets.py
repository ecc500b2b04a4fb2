"""Marker offsets of the refinement where its scan has edges: counts of one
workgroup, of a last 16-byte word that is not full, and of more than one round.
Markers come in triangle order, level + 1 of each: whole numbers, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntri", [1, 256 * 3 + 1, 256 * 5, 256 * 4096, 256 * 4096 + 257, 256 * 9001 + 3])
def test_offsets(ntri):
    import torch
    from paper_1805_01113_amd import mls, workloads as W
    mls.load()
    ctx = mls.Context([W.uniform_faces(64)] * 3, [True] * 3)
    g = torch.Generator(device="cuda").manual_seed(ntri)
    nvert = 4096
    v = torch.rand((3, nvert), generator=g, device="cuda") * 0.02 + 0.4
    tri = torch.randint(0, nvert, (ntri, 3), generator=g, device="cuda", dtype=torch.int32)
    r = ctx.refine(tri, v[0].contiguous(), v[1].contiguous(), v[2].contiguous(), ratio=0.7)
    ctx.sync()
    parts = r["level"].to(torch.int64) + 1
    if ntri > 100:
        assert len(torch.unique(parts)) == 4
    assert r["count"] == int(parts.sum())
    want = torch.repeat_interleave(torch.arange(ntri, device="cuda", dtype=torch.int32), parts)
    assert torch.equal(r["parent"], want)
