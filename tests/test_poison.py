"""The outputs that the binding allocates hold no right answer before a kernel
writes them (the fixture poisoned_memory, active in every test)."""
import numpy as np
import pytest


def test_fresh_memory_is_poisoned():
    import torch
    assert torch.isnan(torch.empty(3, dtype=torch.float64)).all()
    assert torch.isnan(torch.empty((2, 5), dtype=torch.float32)).all()
    assert (torch.empty(4, dtype=torch.int32) == -2).all()
    assert (torch.empty((1,), dtype=torch.int64) == -2).all()
    assert (torch.empty(9, dtype=torch.uint8) == 255).all()
    assert (torch.empty_like(torch.zeros(3, dtype=torch.int32)) == -2).all()


@pytest.mark.gpu
def test_binding_takes_poisoned_memory():
    import torch
    from cases import hand_case
    from gpu_util import device_inputs
    from paper_2407_00047_amd import qlm
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pr, pl = hand_case(np.random.default_rng(1), 20, 3, P=5)
    dpr, dpl = device_inputs(pr, pl)
    out = qlm.plans_like(dpl, 20)
    for x in (out.perm, out.qoff, out.evict_bits):
        assert (x == -2).all()
    assert (qlm.workspace(dpr, 5) == 255).all()
    assert (qlm.search_workspace(dpr, 5, 2) == 255).all()
    assert (qlm.fcfs_workspace(dpr, 5, dpr.total_requests) == 255).all()
