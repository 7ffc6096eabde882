"""Lattices of few spanwise nodes against the same flow repeated over a longer span (GPU).

A flow that is periodic in z with nz nodes is the same flow on a lattice of m nz nodes.  The short
lattice goes to the kernels for few spanwise nodes (the row kernel with FP32 storage, rows of 16 or
32 lanes with FP16), the long one to the kernels of 64-lane rows, and the arithmetic of a node is
the same in all of them: states and outlet histories are equal bit for bit, and the means over z
(FP64 sums in another order: up to 72 nodes of either sign, 1e-13 of the largest) agree.  The inlet
modes have no spanwise wave number, so that the inlet plane is periodic too.

The same lattice with and without sampling likewise, where the two take different kernels."""
import numpy as np
import pytest
import torch

from paper_2304_04214_amd.channel import Channel
from parity_cases import Case, rel_linf

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BOUNDS = {
    "open-slip-sponge": dict(ywall="slip", xbc="inflow", wall_model=True, sponge_cells=3, sponge_nu=0.02),
    "open-bounceback-musker": dict(ywall="bounceback", xbc="inflow", wall_model=True, wall_law="musker",
                                   outlet="zero-gradient"),
    "closed-bounceback-force": dict(ywall="bounceback", xbc="periodic", wall_model=True, g=(2e-5, -1e-5, 5e-6)),
    "periodic-force": dict(ywall="periodic", xbc="periodic", wall_model=False, g=(2e-5, -1e-5, 5e-6), tau0=0.53),
}


def flow(shape, storage, reference, kw):
    """A channel whose inlet modes do not vary in z."""
    c = Case(*shape, storage=storage, reference=reference, **kw)
    if kw["xbc"] == "inflow":
        mt = dict(c.mt)
        mt["d"] = np.array(mt["d"])
        mt["d"][2] = 0.0
        c.ch.set_stg(mt, c.U_g, c.R, c.ab, c.boy, want_fluct=True)
    return c.ch


def outputs(ch, kw, steps, planes):
    ch.stats_attach(planes)
    ch.step(steps)
    means, n = ch.stats_read()
    assert n == steps
    wall = ch.stats_read_wall()[0] if kw["wall_model"] else None
    return ch.populations(), ch.state()[1].clone(), means, wall


@pytest.mark.parametrize("bounds", list(BOUNDS))
@pytest.mark.parametrize("storage,nx,ny,nz,m", [
    # row kernel: 16-lane sums of 16, 9 and 12 nodes, 32-lane sums of 32 and (long enough a launch) 24
    ("f32", 6, 9, 16, 4), ("f32", 7, 10, 9, 8), ("f32", 6, 13, 12, 6), ("f32", 6, 9, 32, 2), ("f32", 404, 12, 24, 3),
    # fused FP16 kernel: 16 and 32 lanes a row, full and in part
    ("f16dev", 6, 9, 16, 4), ("f16dev", 5, 4, 1, 64), ("f16dev", 6, 9, 17, 4), ("f16dev", 7, 13, 32, 2),
    ("f16ref", 6, 9, 16, 4), ("f16ref", 6, 10, 20, 4)])
def test_a_repeated_span_gives_the_same_flow(storage, nx, ny, nz, m, bounds):
    print("repeated span", storage, nx, ny, nz, m, bounds, flush=True)
    kw, ref = BOUNDS[bounds], storage == "f16ref"
    short, long = (flow((nx, ny, n), "f32" if storage == "f32" else "f16dev", ref, kw) for n in (nz, m * nz))
    f = short.populations()
    short.load_populations(f)  # both are encoded from the same numbers
    long.load_populations(torch.cat([f] * m, -1))
    long.state()[1].copy_(torch.cat([short.state()[1]] * m, -1))
    planes, steps = [0, 2, nx - 1], 7
    a, b = outputs(short, kw, steps, planes), outputs(long, kw, steps, planes)
    assert torch.equal(torch.cat([a[0]] * m, -1), b[0])
    if kw["xbc"] == "inflow":
        assert torch.equal(torch.cat([a[1]] * m, -1), b[1])
    for k in range(9):
        assert np.abs(b[2][:, :, k]).max() > 0
        assert rel_linf(a[2][:, :, k], b[2][:, :, k]) <= 1e-13, k
    if kw["wall_model"]:
        assert np.all(b[3] > 0) and rel_linf(a[3], b[3]) <= 1e-13


@pytest.mark.parametrize("bounds", list(BOUNDS))
@pytest.mark.parametrize("nx,ny,nz", [(4, 130, 1), (5, 70, 2), (10, 20, 4), (9, 21, 20), (8, 30, 24)])
def test_sampled_and_other_steps_are_the_same(nx, ny, nz, bounds):
    """Small lattices whose sampled steps go to the general kernel, the others to the row kernel."""
    print("sampled or not", nx, ny, nz, bounds, flush=True)
    kw = BOUNDS[bounds]
    ch = flow((nx, ny, nz), "f32", False, kw)
    f0, h0 = [t.clone() for t in ch.state()]
    out = []
    for sampled in (False, True):
        ch.set_state(f0, h0, 0)
        if sampled:
            ch.stats_attach([0, 2])
        ch.step(9)
        out.append((ch.populations(), ch.state()[1].clone()))
    assert torch.equal(out[0][0], out[1][0])
    if kw["xbc"] == "inflow":
        assert torch.equal(out[0][1], out[1][1])
