"""The inlet plane at times so large that a mode's phase omega t has many more bits than its turns,
against the FP64 oracle of the phases reduced by fmod.

Modes without a wall-normal wave number, and no phase of their own: at these times both would be
rounded away.  Then the plane at t is the plane at 0 with phases fmod(omega t, 2 pi).  Tolerance:
that of the plane against the oracle at ordinary times, 1e-5 of its largest velocity."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_cases import Case

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# one, two and four rows a block
@pytest.mark.parametrize("ny,nz", [(10, 70), (300, 70), (1400, 190)])
@pytest.mark.parametrize("t", [1e18, 3e30, 1e200])
def test_planes_at_far_times(ny, nz, t):
    print("far phases", ny, nz, t, flush=True)
    c = Case(3, ny, nz, ywall="slip", xbc="inflow", wall_model=False, n_modes=40, u_tau=0.004)
    mt = {k: np.array(v, dtype=np.float64) for k, v in c.mt.items()}
    mt["d"][1] = 0.0
    mt["phi"][:] = 0.0
    mt["omega"] = np.where(np.abs(mt["omega"]) < 1e-3, 1e-3, mt["omega"])
    c.ch.set_stg(mt, c.U_g, c.R, c.ab, c.boy, want_fluct=True)
    u = c.ch.stg_fill(t).cpu().numpy()
    c.ch.sync()
    phi = np.fmod(mt["omega"] * t, 2 * np.pi)
    stg = O.StgInputs(mt["q"], mt["sigma"], mt["kmag"], mt["d"], phi, 0.0 * phi, c.U_or, c.R, c.ab, c.boy)
    st, ref, _ = O.stg_plane(c.ocfg, stg, 0.0, want_fluct=True)
    assert st == O.OK
    assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max()
