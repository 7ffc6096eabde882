"""FP16 storage on lattices of few spanwise nodes against the FP64 oracle: outlet history, second
moments and wall statistics, which the short rows reduce by code of their own.

Tolerances: populations and the outlet history 2e-4 of max f as the other FP16 parity tests; with
them a velocity, a difference of populations, is off by at most that much, and a product of two by
twice that times the largest speed; wall statistics 2e-3 as with 64-lane rows."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_cases import Case, rel_linf

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL16, TOL_WALL = 2e-4, 2e-3


@pytest.mark.parametrize("avg", ["local", "line"])
@pytest.mark.parametrize("reference", [False, True])
@pytest.mark.parametrize("shape,kw", [
    ((9, 10, 16), dict(ywall="slip")), ((9, 10, 17), dict(ywall="bounceback")), ((9, 10, 32), dict(ywall="slip")),
    ((7, 9, 5), dict(ywall="slip", wall_law="musker")), ((6, 13, 20), dict(ywall="slip", sponge_cells=3,
                                                                           sponge_nu=0.02)),
    # short rows beyond the caches: every step's stores non-temporal
    ((640, 100, 20), dict(ywall="slip"))])
def test_fp16_histories_moments_and_wall_statistics(shape, kw, reference, avg):
    print("few spanwise nodes", shape, kw, reference, avg, flush=True)
    steps = 12 if shape[0] < 100 else 3
    c = Case(*shape, storage="f16dev", reference=reference, xbc="inflow", wall_model=True, wall_avg=avg, **kw)
    planes = [0, 4, shape[0] - 1]
    c.ch.stats_attach(planes)
    c.ch.step(steps)
    means, n = c.ch.stats_read()
    wall, m = c.ch.stats_read_wall()
    assert n == m == steps
    acc, wacc = np.zeros((len(planes), shape[1], 9)), np.zeros((2, shape[0]))
    st, f, hist = O.run(c.ocfg, c.f_or, c.hist_or, 0, steps, stg=c.stg_or, planes=planes, acc=acc, wall_acc=wacc)
    assert st == O.OK
    f_g, hist_g = c.gpu_state()
    fmax = np.abs(f).max()
    assert rel_linf(f_g, f) <= TOL16 and np.abs(hist_g - hist).max() <= TOL16 * fmax
    ref = acc / (shape[2] * steps)
    assert np.abs(means[:, :, :3] - ref[:, :, :3]).max() <= TOL16 * fmax
    speed = np.sqrt(np.abs(ref[:, :, 3:6]).max()) + TOL16 * fmax
    assert np.abs(means[:, :, 3:] - ref[:, :, 3:]).max() <= 2 * TOL16 * fmax * speed
    ref_w = wacc / (shape[2] * steps)
    assert np.abs(wall - ref_w).max() <= TOL_WALL * np.abs(ref_w).max()
