"""How many states a gradient run keeps (no GPU): what fits a share of the memory that its checkpoints,
its recompute buffers and its adjoint fields leave, so that a run which fits without kept states
fits with them."""
import math
from types import SimpleNamespace

import pytest
import torch

from paper_2304_04214_amd.adjoint import KEEP_SHARE, StatsGradient


def gradient_run(monkeypatch, T, free, dtype=torch.float32, held=0):
    """A run on a 4 x 1 x 8 lattice of one brick a row, `free` bytes on the card, `held` in torch's cache."""
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda dev=None: (free - held, free))
    monkeypatch.setattr(torch.cuda, "memory_reserved", lambda dev=None: held)
    monkeypatch.setattr(torch.cuda, "memory_allocated", lambda dev=None: 0)
    f = torch.zeros((4, 1, 8, 19, 64), dtype=dtype)
    h = torch.zeros((5, 8, 64))
    ch = SimpleNamespace(ny=8, nz=64, state=lambda: (f, h), time=0)
    return StatsGradient(ch, [1], T), f.nbytes + h.nbytes + 6 * 4 * 8 * 64, 2 * (f.numel() * 4 + h.nbytes)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("T", [1, 2, 30, 400, 2000])
@pytest.mark.parametrize("room", [0.5, 0.99, 1.0, 1.01, 1.2, 3.0, 50.0])
def test_a_run_that_fits_without_kept_states_fits_with_them(T, room, dtype, monkeypatch):
    seg = max(1, round(math.sqrt(T)))
    _, state, fields = gradient_run(monkeypatch, T, 1, dtype)
    without = (-(-T // seg) + max(seg - 1, 1)) * state + fields  # checkpoints, recompute ring, adjoint fields
    free = int(room * without)
    run, _, _ = gradient_run(monkeypatch, T, free, dtype, held=free // 3)
    n = min(T - 1, run._keep_states())
    assert n >= 0
    if n == 0:
        assert T == 1 or KEEP_SHARE * (free - without) < state
        return
    left = T - n - 1  # steps before the kept ones
    rest = (-(-left // seg) + 1 + (max(seg - 1, 1) if left else 0)) * state + fields
    assert n * state + rest <= free
    assert n * state <= KEEP_SHARE * free
