"""Host: which spreading takes two launches through the staging buffer and which
one launch per colour, on both sides of the lines that measurements drew: few
tiles with markers against many, few tiles that could hold some against many,
the size of the buffer."""
import pytest

from recorder import run

_CODE = """
def faces(n):
    return [W.uniform_faces(n[d], n[d] / n[0]) for d in range(3)]
result = []
for n, tile, count in %s:
    ctx = mls.Context(faces(n), [True] * 3, spread_tile=tile)
    rec.clear()
    st = L.mls_spread(ctx.h, count, *([ptr] * 9), None)
    names = [k for k, _, _ in rec.launches()]
    grid = [g for k, g, _ in rec.launches() if k in ("k_spread_stage", "k_spread_merge")]
    result.append([st, names.count("k_spread_stage"), names.count("k_spread_merge"), names.count("k_spread_colour"), grid])
    ctx.close()
"""

# cells, tile edge, markers -> colours (0: two launches)
CASES = [
    ((64, 64, 64), 8, 5120, 0),            # one sphere
    ((96, 96, 96), 8, 105984, 0),          # 1104 tiles with markers and 96 for the 1728 there are: 1200
    ((96, 96, 96), 8, 106080, 8),
    ((96, 96, 96), 8, 233280, 8),          # packed: every tile holds markers
    ((128, 128, 128), 8, 64000, 0),
    ((128, 128, 128), 8, 703040, 8),
    ((120, 120, 120), 8, 256000, 0),       # 27 launches are worth more
    ((144, 144, 144), 8, 4201, 0),         # the buffer holds 4201 of the 5832 tiles' boxes
    ((144, 144, 144), 8, 4202, 8),
    ((96, 96, 96), 4, 4000, 0),
    ((96, 96, 96), 4, 16000, 8),           # 13824 tiles that could hold markers
    ((16, 16, 16), 8, 1000, 1),            # one tile: nothing to save
]


def test_route_of_a_spreading(tmp_path):
    out = run(tmp_path, _CODE % ([c[:3] for c in CASES],))
    for (n, tile, count, colours), got in zip(CASES, out):
        assert got[0] == 0
        assert got[1:4] == ([1, 1, 0] if colours == 0 else [0, 0, colours]), (n, tile, count, got)
        if colours == 0:
            tiles = 1
            for v in n:
                tiles *= v // tile
            assert got[4] == [3 * min(tiles, count)] * 2
