"""The FP16 step of the Re_tau = 5200 workload (1536 x 128 x 384, deviations from the weights) goes out
as one bulk dispatch per range of x-planes: one step against the FP64 oracle on nodes of both planes
at every border between them, with the tolerance of the other FP16 parity tests."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_cases import rel_linf
from test_gpu_fullsize import workload

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def test_nodes_on_both_sides_of_every_bulk_range():
    print("bulk ranges", flush=True)
    cfg, stg, f, hist, ch, planes = workload("c3", "f16dev", full_pert=False)
    n, per = ch.timed_dispatches()
    assert (n, per) == (5, 308)
    nx, ny, nz = cfg.nx, cfg.ny, cfg.nz
    xs = sorted({1, nx - 2} | {k * per + d for k in range(1, n) for d in (-2, -1, 0, 1)})
    g = np.random.default_rng(5)
    ys = [0, 1, 2, 3, 4, ny // 2, ny - 5, ny - 2, ny - 1, *g.integers(0, ny, 12)]
    zs = [0, 1, 63, 64, nz - 1, *g.integers(0, nz, 12)]
    nodes = np.unique([(x * ny + y) * nz + z for x in xs for y in ys for z in zs]).astype(np.int64)
    ch.step(1)
    ch.sync()
    gpu = ch.populations().reshape(19, -1)[:, torch.as_tensor(nodes, device="cuda")].cpu().numpy()
    st, ref, _ = O.step_nodes(cfg, f, hist, 1.0, nodes, stg=stg)
    assert st == O.OK
    assert rel_linf(gpu.astype(np.float64), ref) <= 2e-4
