"""Each step of lbm_step_keep and lbm_step_record reads its own inlet plane, whatever buffers the
caller gives for them: a buffer may come back as long as neighbours differ, and a launch fills
several planes before the first of their steps runs.  On a host double of the HIP runtime (no GPU),
which replays the fills and the reads in the order of the stream."""
import pytest

from host_double import double

CODE = """
R = Runtime()
A, L = R.A, R.L
entry, n, us, fs, storage = %r
h = R.channel(5, 9, 16, storage=storage, xbc=1)
word = lambda p, i: C.cast(p, C.POINTER(C.c_uint64))[i]
held, out = {}, dict(races=[], reads=[], fills=[])

def on_launch(kernel, args):
    grid = R.launches[-1][1]
    if kernel == "stg_fill_kernel":
        t = C.cast(args[4], C.POINTER(C.c_double))[0]
        dst = [word(args[9], j) for j in range(64)]
        bufs = [(dst[j], t + j) for j in range(grid[2])] + [(dst[32 + j], t + j) for j in range(grid[2])]
        out["fills"].append(grid[2])
        out["races"] += [b for b, _ in bufs if [c for c, _ in bufs].count(b) > 1]
        held.update(bufs)
    elif kernel.startswith("collide_"):
        out["reads"].append(held.get(word(args[0], 4)))  # CollideArgs::u_in

R.on_launch = on_launch
f, hist = R.array(range(1000, 1000 + n)), R.array(range(2000, 2000 + n))
u, fl = R.array([3000 + k for k in us]), R.array([4000 + k for k in fs])
out["status"] = (L.lbm_step_keep(h, None, n, f, hist, u, fl) if entry == "keep" else
                 L.lbm_step_record(h, None, R.plane(0), R.plane(2), 0.0, n, f, hist, u, fl))
emit(out)
"""


@pytest.mark.parametrize("entry", ["keep", "record"])
@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,period,batches", [
    (5, 5, [5]), (70, 70, [32, 32, 6]),  # buffers of their own
    (6, 2, [2, 2, 2]), (7, 3, [3, 3, 1]), (66, 33, [32, 32, 2]), (64, 31, [31, 31, 2])])
def test_every_step_reads_its_own_inlet_plane(entry, storage, n, period, batches, tmp_path):
    ks = [k % period for k in range(n)]
    out = double(CODE % ((entry, n, ks, ks, storage),), tmp_path)
    assert out["status"] == 0
    assert out["races"] == []
    assert out["reads"] == [k + 1.0 for k in range(n)]
    assert out["fills"] == batches


def test_planes_and_fluctuations_may_trade_buffers(tmp_path):
    """uin_keep[1] is fluct_keep[0]: the second plane comes from a launch of its own."""
    out = double(CODE % (("keep", 3, [0, 1000, 1], [0, 5, 6], 0),), tmp_path)
    assert out["status"] == 0 and out["races"] == [] and out["reads"] == [1.0, 2.0, 3.0]
    assert out["fills"] == [1, 2]


FORBIDDEN = """
R = Runtime()
A, L = R.A, R.L
h = R.channel(5, 9, 16, storage=%r, xbc=1)
bytes_ = 4 * 3 * 9 * 16
f, hist = R.array([1000, 1001]), R.array([2000, 2001])
def planes(**at):
    u, fl = [R.plane(3000 + k).value for k in range(3)], [R.plane(4000 + k).value for k in range(3)]
    for k, v in at.items():
        (u if k[0] == "u" else fl)[int(k[1])] = v
    return (C.c_void_p * 3)(*u), (C.c_void_p * 3)(*fl)
own = R.plane(3001).value
bad = dict(u_equal_neighbours=dict(u1=R.plane(3000).value), f_equal_neighbours=dict(f2=R.plane(4001).value),
           u_is_f=dict(f1=own), u_overlaps_f=dict(f1=own + bytes_ - 4), f_overlaps_u=dict(f1=own - 64),
           u_bound=dict(u0=R.u_in), u_bound_fluct=dict(u1=R.fluct), f_bound=dict(f2=R.fluct),
           f_bound_u=dict(f0=R.u_in), u_overlaps_bound=dict(u2=R.u_in + 16), u_null=dict(u1=None), f_null=dict(f1=None))
out = {k: L.lbm_step_keep(h, None, 3, f, hist, *planes(**v)) for k, v in bad.items()}
# inputs given with the call are the bound ones
s = A.Stg.from_buffer_copy(R.stg)
s.u_in = R.plane(500).value
out["u_given"] = L.lbm_step_keep(h, C.byref(s), 3, f, hist, *planes(u1=R.plane(500).value))
none = len(R.launches)
out2 = dict(next_to_f=L.lbm_step_keep(h, None, 3, f, hist, *planes(f1=own + bytes_)),
            formerly_bound=L.lbm_step_keep(h, C.byref(s), 3, f, hist, *planes(u1=R.u_in)))
emit([out, none, out2])
"""


@pytest.mark.parametrize("storage", [0, 1])
def test_forbidden_plane_buffers_are_rejected(storage, tmp_path):
    from paper_2304_04214_amd import _abi as A
    bad, launches, good = double(FORBIDDEN % storage, tmp_path)
    assert bad == {k: A.LBM_ERR_ARG for k in bad} and launches == 0
    assert good == {k: A.LBM_OK for k in good}
