"""Host: the queue of gradient pairs that a second kernel redoes.  That kernel
returns the queue's counts to zero, so a call launches two kernels; where a
launch failed the counts are unknown, and the next call has to clear them."""
import pytest

from recorder import run

_CODE = """
ctx = mls.Context([W.uniform_faces(16)] * 3, [True] * 3)
def interp(n):
    return L.mls_interp_grad(ctx.h, n, *([ptr] * 8), None, None, None, None)
def build(n):
    return L.mls_build_grad(ctx.h, n, ptr, ptr, ptr, 0, ptr, ptr, ptr, None)
call = %s
result = []
for n, bad in %s:
    rec.clear()
    if bad: rec.fail(bad)
    st = call(n)
    result.append([st, [k for k, _, _ in rec.launches()]])
"""


@pytest.mark.parametrize("call,first,second", [("interp", "k_interp_grad", "k_interp_grad_fp64"),
                                               ("build", "k_build_grad", "k_build_grad_fp64")])
def test_counts_are_cleared_after_a_failed_launch(tmp_path, call, first, second):
    both = [first, second]
    out = run(tmp_path, _CODE % (call, [(100, ""), (100, ""), (100, second), (100, ""), (50, ""), (200, ""),
                                        (10, first + "I" if call == "interp" else first + "E"), (200, ""), (200, "")]))
    assert out[0] == [0, ["k_queue_clear"] + both]     # first use
    assert out[1] == [0, both]
    assert out[2] == [-5, [first]]                     # entries without the kernel that takes them
    assert out[3] == [0, ["k_queue_clear"] + both]
    assert out[4] == [0, both]
    assert out[5] == [0, ["k_queue_clear"] + both]     # growth
    assert out[6][0] == -5
    assert out[7] == [0, ["k_queue_clear"] + both]
    assert out[8] == [0, both]
