"""FP16 storage on lattices of at most 32 and at most 16 spanwise nodes (two and four rows a wave in
the fused kernel): fields and statistics against the FP64 oracle.

Tolerance: that of the other FP16 parity tests, 2e-4 of max f after 20 steps (half-ulp roundings of
deviations below 2^-6, 2^-18 each, about 20 of them); velocities are differences of the same
populations, so their means are held to the same absolute error."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_cases import Case, rel_linf

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL16 = 2e-4


@pytest.mark.parametrize("reference", [False, True])
@pytest.mark.parametrize("shape,kw", [
    ((6, 9, 32), dict(ywall="slip", xbc="inflow", wall_model=True)),
    ((5, 4, 17), dict(ywall="bounceback", xbc="inflow", wall_model=True)),
    ((6, 13, 16), dict(ywall="slip", xbc="inflow", wall_model=True, sponge_cells=3, sponge_nu=0.02)),
    ((5, 10, 1), dict(ywall="slip", xbc="inflow", wall_model=True)),
    ((5, 7, 20), dict(ywall="periodic", xbc="periodic", wall_model=False, g=(2e-5, -1e-5, 5e-6), tau0=0.53)),
    ((5, 11, 9), dict(ywall="bounceback", xbc="periodic", wall_model=True, wall_avg="line", g=(1e-5, 0.0, 0.0))),
    # non-temporal stores with short rows, cached stores with 64-lane rows
    ((622, 100, 3), dict(ywall="slip", xbc="inflow", wall_model=True)),
    ((190, 64, 40), dict(ywall="slip", xbc="inflow", wall_model=True)),
])
def test_fp16_fields_and_statistics_match_the_oracle(shape, kw, reference):
    print("short rows", shape, kw, reference, flush=True)
    c = Case(*shape, storage="f16dev", reference=reference, **kw)
    planes = [0, 2, shape[0] - 1]
    c.ch.stats_attach(planes)
    c.ch.step(20)
    means, n = c.ch.stats_read()
    assert n == 20
    st, f_or, _, acc = c.run_oracle(20, planes=planes)
    assert st == O.OK
    f_g, _ = c.gpu_state()
    assert rel_linf(f_g, f_or) <= TOL16
    ref = acc / (shape[2] * 20)
    assert np.abs(means[:, :, :3] - ref[:, :, :3]).max() <= TOL16 * np.abs(f_or).max()
