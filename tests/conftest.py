import os
import sys

import pytest

_ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_TESTS = os.path.dirname(os.path.abspath(__file__))
for p in (_ROOT, _TESTS):
    if p not in sys.path:
        sys.path.insert(0, p)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long CPU test")


@pytest.fixture(scope="session")
def orc():
    import oracle
    return oracle.default()


@pytest.fixture(autouse=True)
def poisoned_memory(monkeypatch):
    """torch.empty and torch.empty_like, from which the binding takes outputs and
    workspaces, give memory that no right answer holds: NaN, -2, and bytes of 255
    (a workspace's doubles are then NaN and its integers -1).  Fresh memory is often
    the block that held the last right answer, so that an entry which a kernel leaves
    unwritten would pass."""
    import torch

    def poison(make):
        def made(*args, **kwargs):
            t = make(*args, **kwargs)
            if t.is_floating_point():
                t.fill_(float("nan"))
            elif t.dtype != torch.bool:
                t.fill_(255 if t.dtype == torch.uint8 else -2)
            # (the call that takes it may run on another stream)
            if t.is_cuda and not torch.cuda.is_current_stream_capturing():
                torch.cuda.current_stream(t.device).synchronize()
            return t
        return made

    monkeypatch.setattr(torch, "empty", poison(torch.empty))
    monkeypatch.setattr(torch, "empty_like", poison(torch.empty_like))
