"""Attaching statistics planes, on a host double of the HIP runtime (no GPU): planes that are attached
already keep their buffers and block lists, others get new ones, and a stream under capture is
refused either way (the call is not for a graph: on a replay it would not start the count again)."""
import pytest

from host_double import double

CODE = """
R = Runtime()
A, L = R.A, R.L
h = R.channel(9, 9, 16, storage=%r, xbc=1, wall_model=1)
def attach(*planes):
    R.calls.clear()
    arr = (C.c_int32 * len(planes))(*planes)
    st = L.lbm_stats(h, A.STATS_ATTACH, arr, len(planes), None, None)
    return [st, sorted({c[0] for c in R.calls})]
out = [attach(2, 5), attach(2, 5), attach(5, 2), attach(5, 2)]
assert L.lbm_step(h, None, 3) == A.LBM_OK
R.dev.double_capturing(1)
out += [attach(5, 2), attach(5, 3)]
R.dev.double_capturing(0)
n, host = C.c_int64(), (C.c_double * (2 * 9 * 9))()
assert L.lbm_stats(h, A.STATS_READ, None, 0, host, C.byref(n)) == A.LBM_OK
emit([out, n.value])
"""


@pytest.mark.parametrize("storage", [0, 1])
def test_attach_again_and_under_capture(storage, tmp_path):
    from paper_2304_04214_amd import _abi as A
    out, samples = double(CODE % storage, tmp_path)
    assert [st for st, _ in out] == [A.LBM_OK] * 4 + [A.LBM_ERR_HIP] * 2
    assert "hipMalloc" in out[0][1] and out[1][1] == ["hipMemsetAsync"]
    assert "hipMalloc" in out[2][1] and out[3][1] == ["hipMemsetAsync"]
    for _, calls in out[4:]:  # refused before anything is recorded or freed
        assert not {"hipMemsetAsync", "hipMemcpyAsync", "hipMalloc", "hipFree"} & set(calls)
    assert samples == 3  # the refused calls change nothing
