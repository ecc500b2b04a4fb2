"""The two shortcuts of the cell lookup, in the device's arithmetic on the CPU,
against the plain rule faces[i] <= x < faces[i+1].

FP32 lookup on a uniform axis: t = (x - t_off) t_scale in FP32; where its
fraction is further than t_eps from 0 and 1, its floor must be the cell.
Buckets of a stretched axis: the cell of x must be among the cells of its
bucket, and buckets must stay small.
"""
import numpy as np
import pytest

from paper_1805_01113_amd import workloads as W

ULP = 2.0 ** -24


def _near(r, faces, count):
    """FP32 coordinates: uniform over the axis, and within a few FP32 steps of the faces."""
    x = r.uniform(faces[0], faces[-1], count).astype(np.float32)
    f = r.choice(faces, count).astype(np.float32)
    for _ in range(3):
        f = np.where(r.random(count) < 0.5, np.nextafter(f, np.float32(-np.inf)), np.nextafter(f, np.float32(np.inf)))
    x = np.concatenate([x, f, faces.astype(np.float32)])
    return x[(x.astype(np.float64) >= faces[0]) & (x.astype(np.float64) < faces[-1])]


@pytest.mark.parametrize("n,length,origin", [(3, 1.0, 0.0), (64, 1.0, 0.0), (517, 2.2, -3.7), (1000, 0.125, 0.0),
                                             (2048, 6.2831853, 0.0), (300, 1.0, 1000.0), (1024, 1.0, 1e-3)])
def test_fp32_cell_of_a_uniform_axis(n, length, origin):
    r = np.random.default_rng(n)
    f = W.uniform_faces(n, length, origin)
    L = f[-1] - f[0]
    inv_h = n / L
    dev = np.abs(f - (f[0] + np.arange(n + 1) * (L / n))).max()
    eps = 1.01 * ULP * (abs(f[0]) * inv_h + 4.0 * n) + dev * inv_h + 1e-6
    x = _near(r, f, 200000)
    t = (x - np.float32(f[0])) * np.float32(inv_h)
    fr = t - np.floor(t)
    e = np.float32(eps if eps < 0.25 else 1.0)
    sure = (fr > e) & (fr < np.float32(1.0) - e) & (t > 0) & (t < n)
    cell = np.searchsorted(f, x.astype(np.float64), side="right") - 1
    assert np.array_equal(np.floor(t[sure]).astype(np.int64), cell[sure])
    # face nodes: centres[i - 1] <= x < centres[i]
    th = t + np.float32(0.5)
    fr = th - np.floor(th)
    sf = (fr > e) & (fr < np.float32(1.0) - e) & (t > 0) & (t < n)
    node = np.searchsorted(0.5 * (f[:-1] + f[1:]), x.astype(np.float64), side="right")
    assert np.array_equal(np.floor(th[sf]).astype(np.int64), node[sf])
    if eps < 0.01:      # a shortcut: nearly every coordinate away from the faces takes it
        assert sure[:200000].mean() > 0.95


@pytest.mark.parametrize("faces", [W.tanh_faces(768, 1.5, 2.5), W.tanh_faces(7, 1.0, 1.2),
                                   W.tanh_faces(2048, 3.0, 3.5) - 1.5,
                                   np.concatenate([[0.0], np.cumsum(1.02 ** np.arange(200))])])
def test_buckets_of_a_stretched_axis(faces):
    r = np.random.default_rng(len(faces))
    n, f0 = len(faces) - 1, faces[0]
    nb = 4 * n
    scale = nb / (faces[-1] - f0)

    def of(X):
        return np.clip(((X - f0) * scale).astype(np.int64), 0, nb - 1)

    bf = of(faces)
    first, last = np.empty(nb, dtype=np.int64), np.empty(nb, dtype=np.int64)
    k = 0
    for b in range(nb):
        while k < n - 1 and bf[k + 1] < b:
            k += 1
        q = k
        while q < n - 1 and bf[q + 1] <= b:
            q += 1
        first[b], last[b] = k, q
    x = np.concatenate([_near(r, faces, 100000).astype(np.float64), faces[:-1], np.nextafter(faces[1:], -np.inf)])
    cell = np.searchsorted(faces, x, side="right") - 1
    b = of(x)
    assert np.all((first[b] <= cell) & (cell <= last[b]))
    assert (last[b] - first[b]).mean() < 6.0
