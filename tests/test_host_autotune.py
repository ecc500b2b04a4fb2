"""Host: the autotuner times a shape only where it changes a launch, and a result
found on one route of the spreading is not served to marker counts on the
other.  The recording runtime reports times that differ by chance only, so any
pick among equal launches would be by chance too."""
import json

import pytest

from recorder import run

_CODE = """
result = []
for n, tile, count, cache in %s:
    ctx = mls.Context([W.uniform_faces(n)] * 3, [True] * 3)
    before = ctx.tune_get()
    rec.clear()
    b = step_buffers(count)
    r = mls._TuneReport()
    st = L.mls_autotune(ctx.h, mls.MLS_EXACT, mls.MLS_STEP_COMPACT, ctypes.byref(b), cache.encode() or None, ctypes.byref(r), None)
    shapes = [(k, g, t) for k, g, t in rec.launches() if k in ("k_build_interp", "k_spread_stage", "k_spread_colour")]
    result.append([st, before, ctx.tune_get(), r.from_cache, r.candidates, shapes])
    ctx.close()
"""


def _tune(tmp_path, runs):
    return run(tmp_path, _CODE % ([(n, 0, c, cache) for n, c, cache in runs],))


@pytest.mark.parametrize("n,count", [(64, 5120), (48, 1000)])
def test_shapes_without_effect_stay(tmp_path, n, count):
    st, before, after, cached, cand, shapes = _tune(tmp_path, [(n, count, "")])[0]
    assert st == 0 and not cached
    assert {k for k, _, _ in shapes} == {"k_build_interp", "k_spread_stage"}
    # every tiling of this box is spread in two launches and every build grid is the same
    tilings = {64: 3, 48: 5}[n]            # edges 4, 8, 16; 4, 6, 8, 12, 16
    assert cand == 1 + 4 + tilings
    for k in ("spread_blocks_per_cu", "spread_threads", "build_blocks_per_cu"):
        assert after[k] == before[k]


def test_shapes_with_effect_are_timed(tmp_path):
    st, _, after, _, cand, shapes = _tune(tmp_path, [(512, 20 * 10 ** 6, "")])[0]
    assert st == 0
    assert {k for k, _, _ in shapes} == {"k_build_interp", "k_spread_colour"}
    builds = [g for k, g, _ in shapes if k == "k_build_interp"]
    assert {2064, 4104, 8208, 16392} <= set(builds)
    assert {t for k, _, t in shapes if k == "k_spread_colour"} == {128, 192, 256}
    assert cand > 4 + 4 + 3 * 3 * 3


def test_a_result_is_not_served_across_the_routes(tmp_path):
    cache = str(tmp_path / "tune.jsonl")
    # one octave of marker counts: the boxes of 4201 tiles of 8 cells fit the buffer, those of 8000 do not
    out = _tune(tmp_path, [(256, 4150, cache), (256, 8000, cache), (256, 4180, cache), (256, 7900, cache)])
    assert [o[3] for o in out] == [0, 0, 1, 1]
    with open(cache) as f:
        keys = [json.loads(line)["key"] for line in f]
    assert len(set(keys)) == 2
    # where no tiling is spread in two launches the key is the one that older files hold
    plain = str(tmp_path / "plain.jsonl")
    out = _tune(tmp_path, [(512, 10 ** 6, plain)])
    with open(plain) as f:
        assert json.loads(f.readline())["key"] == "unknown|cu256|512x512x512|p111|s-1|m0|f1|n19"
