"""Steps that keep their states for the adjoint sweep, against the same steps without: the kernels
and their order are those of lbm_step and of the recompute, so states, planes, statistics and
gradients are equal bit for bit."""
import numpy as np
import pytest
import torch

from paper_2304_04214_amd import _abi as A
from paper_2304_04214_amd.adjoint import StatsGradient
from parity_cases import Case

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

OPEN = dict(ywall="slip", xbc="inflow", wall_model=True)
CLOSED = dict(ywall="bounceback", xbc="periodic", wall_model=False, g=(2e-5, 0.0, 0.0))


@pytest.mark.parametrize("storage,nz,n,kw", [
    ("f32", 70, 3, OPEN), ("f32", 20, 35, OPEN), ("f16dev", 70, 4, OPEN), ("f16dev", 16, 1, OPEN),
    ("f16dev", 40, 2, dict(OPEN, wall_avg="line")), ("f32", 40, 2, dict(OPEN, wall_avg="line")),
    ("f32", 33, 5, CLOSED), ("f16dev", 33, 1, CLOSED)])
def test_step_keep_matches_step(storage, nz, n, kw):
    print("keep", storage, nz, n, kw, flush=True)
    ch = Case(8, 8, nz, storage=storage, **kw).ch
    inflow = kw["xbc"] == "inflow"
    f0, h0 = [t.clone() for t in ch.state()]
    t0 = ch.time
    ch.stats_attach([2, 5])
    new = lambda t, m: [torch.empty_like(t) for _ in range(m)]
    plane = torch.empty((3, 8, nz), device="cuda")
    keep = new(f0, n - 1), new(h0, n - 1), new(plane, n), new(plane, n)
    start, start_h = ch.state()
    ch.step_keep(n, *keep)
    valid = torch.ones_like(f0, dtype=torch.bool)  # padding nodes z >= nz are unwritten
    valid[:, -1, ..., (nz - 1) % 64 + 1:] = False
    assert ch.time == t0 + n and torch.equal(start[valid], f0[valid]) and torch.equal(start_h, h0)
    last, last_h = [t.clone() for t in ch.state()]
    bound = [t.clone() for t in (ch.u_in, ch.fluct)] if inflow else None
    means = ch.stats_read()
    ch.set_state(f0, h0, t0)
    ch.stats_reset()
    for k in range(n):
        ch.step(1)
        f, h = ch.state()
        assert torch.equal(f[valid], (keep[0] + [last])[k][valid]), k
        if inflow:
            assert torch.equal(h, (keep[1] + [last_h])[k]), k
            assert torch.equal(ch.u_in, keep[2][k]) and torch.equal(ch.fluct, keep[3][k]), k
    assert not inflow or (torch.equal(bound[0], ch.u_in) and torch.equal(bound[1], ch.fluct))
    again = ch.stats_read()
    assert means[1] == again[1] == n and np.array_equal(means[0], again[0])


@pytest.mark.parametrize("storage,steps,kw", [("f32", 9, OPEN), ("f16dev", 9, OPEN), ("f32", 1, OPEN), ("f32", 4, CLOSED)])
def test_gradients_do_not_depend_on_the_kept_steps(storage, steps, kw):
    print("gradient", storage, steps, kw, flush=True)
    ch = Case(8, 8, 24, storage=storage, **kw).ch
    res = []
    for states in (steps, 3, 1, 0, None):  # None: checkpoints of a given segment
        run = StatsGradient(ch, [2, 5], steps, segment=None if states is not None else 2)
        run._keep_states = lambda: states
        for _ in range(2):  # the second run uses the buffers of the first
            means = run.forward()
            assert ch.time == run.t0 + steps
            res.append((means, ch.populations(), run.backward(means), run.backward(means)))
    for means, f, g, g2 in res:
        assert np.array_equal(means, res[0][0]) and torch.equal(f, res[0][1])
        assert np.array_equal(g, res[0][2]) and np.array_equal(g2, g)


def test_step_keep_rejects_bad_buffers():
    ch = Case(8, 8, 24, storage="f32", **OPEN).ch
    ch.step(1)
    f, h = ch.state()
    fb, hb, u = torch.empty_like(f), torch.empty_like(h), [torch.empty((3, 8, 24), device="cuda") for _ in range(2)]
    for args in [([f], [hb], u, u), ([fb], [h], u, u), ([fb.flatten()[1:]], [hb], u, u)]:
        with pytest.raises(Exception):
            ch.step_keep(2, *args)
    L, n = A.lib(), 2
    assert L.lbm_step_keep(None, None, n, None, None, None, None) == A.LBM_ERR_ARG
    assert L.lbm_step_keep(ch._h, None, n, None, None, None, None) == A.LBM_ERR_ARG
    assert L.lbm_step_keep(ch._h, None, -1, None, None, None, None) == A.LBM_ERR_ARG
    ch.step(1)  # the handle is as it was
    assert ch.time == 2
