import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def vt():
    """The Python binding over the C-ABI library (built beforehand, in-tree)."""
    import paper_2604_09558_amd as pkg
    return pkg


@pytest.fixture(scope="session")
def kernels():
    """kernels(call): names of the HIP kernels that call() launches, template arguments included."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    def names(call):
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            call()
            torch.cuda.synchronize()
        return [e.name for e in prof.events() if str(e.device_type).endswith("CUDA")]
    return names
