"""The row kernel (FP32 storage, nz <= 32): fields, plane statistics and wall statistics against
the FP64 oracle at the edges of its blocks, and its choice by the spanwise extent.

Tolerances: as the other FP32 parity tests, 1e-5 of max f for the populations after 20 steps and
2e-5 of max |u| for velocities (the absolute rounding error of populations of 1/3, about 1e-7,
against flows of max |u| ~ 1e-2); a product of two velocities doubles the relative error, a mean
over z and steps adds none.
"""
import numpy as np
import pytest
import torch

import oracle as O
from parity_cases import Case, rel_linf

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL32, TOL_U = 1e-5, 2e-5

CASES = {
    # nz = 32, 17, 16, 1: 4, 7, 8 and 128 rows fit a block of 128 threads
    "one-block-a-plane": ((6, 4, 32), dict(ywall="slip", xbc="inflow", wall_model=True)),
    "ragged-groups": ((5, 9, 32), dict(ywall="slip", xbc="inflow", wall_model=True)),
    "idle-threads": ((5, 15, 17), dict(ywall="slip", xbc="inflow", wall_model=True, sponge_cells=3, sponge_nu=0.02)),
    "helper-rows": ((4, 19, 16), dict(ywall="bounceback", xbc="inflow", wall_model=True)),
    "one-column": ((4, 130, 1), dict(ywall="slip", xbc="inflow", wall_model=True)),
    "two-columns": ((4, 70, 2), dict(ywall="periodic", xbc="periodic", wall_model=False, g=(2e-5, -1e-5, 5e-6),
                                     tau0=0.53)),
    "bounceback-force": ((5, 21, 20), dict(ywall="bounceback", xbc="periodic", wall_model=False,
                                           g=(1e-5, 0.0, 0.0))),
    "line-averaged": ((5, 11, 24), dict(ywall="slip", xbc="inflow", wall_model=True, wall_avg="line")),
    # above 2^17 nodes: blocks of 256 threads
    "large": ((260, 20, 27), dict(ywall="slip", xbc="inflow", wall_model=True)),
    # the two sides of the number of rows up to which the row kernel is taken
    "most-rows": ((620, 100, 4), dict(ywall="slip", xbc="inflow", wall_model=True)),
    "too-many-rows": ((622, 100, 4), dict(ywall="slip", xbc="inflow", wall_model=True)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fields_and_statistics_match_the_oracle(name):
    shape, kw = CASES[name]
    print("rows", name, shape, flush=True)
    steps = 4 if shape[0] > 100 else 20
    c = Case(*shape, **kw)
    planes = [0, 1, shape[0] - 1]
    c.ch.stats_attach(planes)
    c.ch.step(steps)
    means, n = c.ch.stats_read()
    assert n == steps
    st, f_or, hist_or, acc = c.run_oracle(steps, planes=planes)
    assert st == O.OK
    f_g, hist_g = c.gpu_state()
    assert rel_linf(f_g, f_or) <= TOL32
    if kw["xbc"] == "inflow":
        assert rel_linf(hist_g, hist_or) <= TOL32
    ref = acc / (shape[2] * steps)
    umax = np.abs(ref[:, :, :3]).max()
    assert np.abs(means[:, :, :3] - ref[:, :, :3]).max() <= TOL_U * umax
    assert np.abs(means[:, :, 3:] - ref[:, :, 3:]).max() <= 2 * TOL_U * np.abs(ref[:, :, 3:]).max()
    if kw["wall_model"]:
        wall, _ = c.ch.stats_read_wall()
        assert wall.shape == (2, shape[0]) and np.all(wall > 0)


def test_wall_statistics_equal_those_of_the_line_by_line_kernel():
    """u_tau of the wall rows does not depend on how rows are given to waves: a lattice that repeats
    in z twice over (nz = 32, row kernel; nz = 64, one wave a row) has the same means.  The states
    are equal bit for bit, the FP64 sums over z differ by their order: 64 additions, 1e-14 relative."""
    nx, ny = 6, 9
    got = []
    for nz in (32, 64):
        c = Case(nx, ny, 32, ywall="slip", xbc="periodic", wall_model=True) if nz == 32 else \
            Case(nx, ny, 64, ywall="slip", xbc="periodic", wall_model=True)
        f = got[0][0] if got else c.ch.populations()
        c.ch.load_populations(torch.cat([f, f], -1) if nz == 64 else f)
        c.ch.stats_attach([2])
        c.ch.step(3)
        means, _ = c.ch.stats_read()
        wall, _ = c.ch.stats_read_wall()
        got.append((f, c.ch.populations(), means, wall))
    assert torch.equal(torch.cat([got[0][1]] * 2, -1), got[1][1])
    assert rel_linf(got[0][2], got[1][2]) <= 1e-14
    assert rel_linf(got[0][3], got[1][3]) <= 1e-14
