"""One adjoint step on FP16 states in the kernel that pulls the state non-temporally (lambda buffers
of 225 to 320 MiB: 400 x 64 x 64, the Re_tau = 1000 adjoint workload's parameters), against the FP64
oracle with the tolerances of the other adjoint tests."""
import pytest
import torch

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("storage", ["f16dev", "f16ref"])
def test_adjoint_step_with_nontemporal_pulls(storage, monkeypatch):
    import test_gpu_fullsize as T
    whole = T.workload
    monkeypatch.setattr(T, "workload", lambda name, st: whole(name, st, shape=(400, 64, 64)))
    T.test_full_size_adjoint_step("c4", storage)
