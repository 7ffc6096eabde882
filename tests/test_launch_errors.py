"""A kernel launch that fails is reported by the call that made it, and the handle's time does not
advance, on every route of a step (a host double of the HIP runtime; no GPU)."""
import pytest

from host_double import double

CODE = """
R = Runtime()
A, L = R.A, R.L
shape, kw, kernel = %r, %r, %r
h = R.channel(*shape, **kw)
n = 3
keep = [R.array(range(10 + 20 * k, 10 + 20 * k + n)) for k in range(4)]
calls = dict(step=lambda: L.lbm_step(h, None, n),
             step_keep=lambda: L.lbm_step_keep(h, None, n, *keep),
             step_record=lambda: L.lbm_step_record(h, None, R.plane(0), R.plane(2), 0.0, n, *keep))
t, out = C.c_int64(), {}
for name, call in calls.items():
    R.fail = lambda k: k == kernel
    failed = call()
    L.lbm_get_state(h, None, None, C.byref(t))
    time = t.value
    R.fail = lambda k: False
    out[name] = failed, time, call()
    L.lbm_set_state(h, R.plane(0), R.plane(1), R.plane(2), R.plane(3), 0)
emit([out, sorted({k for k, *_ in R.launches})])
"""

ROUTES = {
    "rows": ((5, 9, 16), dict(storage=0), "collide_rows_kernel"),
    "rows-inflow": ((5, 9, 16), dict(storage=0, xbc=1, wall_model=1), "collide_rows_kernel"),
    "general": ((5, 9, 70), dict(storage=0), "collide_general_kernel"),
    "general-ranges": ((12000, 32, 8), dict(storage=0), "collide_general_kernel"),
    "fused": ((5, 9, 70), dict(storage=1, xbc=1), "collide_fused_kernel"),
    "fused-short-rows": ((5, 9, 16), dict(storage=1), "collide_fused_kernel"),
    "bulk": ((1040, 128, 128), dict(storage=1, xbc=1), "collide_bulk_kernel"),
    "bulk-general": ((1040, 128, 128), dict(storage=1, xbc=1), "collide_general_kernel"),
    "wall-line": ((5, 9, 16), dict(storage=0, wall_model=1, wall_avg=1), "wall_line_kernel"),
    "inlet": ((5, 9, 16), dict(storage=0, xbc=1), "stg_fill_kernel"),
}


@pytest.mark.parametrize("route", list(ROUTES))
def test_a_failed_launch_is_reported(route, tmp_path):
    from paper_2304_04214_amd import _abi as A
    shape, kw, kernel = ROUTES[route]
    out, kernels = double(CODE % (shape, kw, kernel), tmp_path)
    assert kernel in kernels, kernels
    for name, (failed, time, then) in out.items():
        assert failed == A.LBM_ERR_HIP, (name, failed)
        assert time == 0, (name, time)
        assert then == A.LBM_OK, (name, then)
