"""Host: workgroups of the build launches as the marker count and the tunable
number of workgroups per compute unit (256 of them) change."""
import pytest

from recorder import run

_CODE = """
ctx = mls.Context([W.uniform_faces(64)] * 3, [True] * 3)
result = {}
for n in %s:
    for v in %s:
        ctx.tune_set(build_blocks_per_cu=v)
        rec.clear()
        for method in (mls.MLS_EXACT, mls.MLS_FAST):
            assert L.mls_build(ctx.h, n, ptr, ptr, ptr, method, ptr, ptr, None, None) == 0
        result["%%d %%d" %% (n, v)] = [g for k, g, _ in rec.launches() if k in ("k_build_exact", "k_build_fast")]
"""

CUS, WAVES = 256, 4
# markers: one workgroup, around a resident round of 768, far past it, and around the line of 16 items a wavefront
NS = [1, 64 * 1024, 64 * 1024 + 1, 10 ** 6, 350000, 11184768, 11184896, 16 * 10 ** 6, 10 ** 8]
PER_CU = [1, 2, 3, 8, 32, 64]


def test_more_workgroups_per_unit_never_start_fewer(tmp_path):
    got = run(tmp_path, _CODE % (NS, PER_CU))
    for n in NS:
        need = (3 * ((n + 63) // 64) + WAVES - 1) // WAVES
        row = [got["%d %d" % (n, v)] for v in PER_CU]
        for j in range(2):
            grids = [r[j] for r in row]
            assert grids == sorted(grids), (n, grids)
            for v, g in zip(PER_CU, grids):
                assert g % 24 == 0 and g <= (min(need, CUS * v) + 23) // 24 * 24, (n, v, g)
        # the exact build: one resident round below the line, all of the grid past it
        exact = [r[0] for r in row]
        if need <= 768 or need >= 16 * CUS * 32:
            assert exact == [(min(need, CUS * v) + 23) // 24 * 24 for v in PER_CU]
        else:
            assert exact == [(min(768, CUS * v) + 23) // 24 * 24 for v in PER_CU]
