import functools
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: long-running CPU check")


@pytest.fixture(scope="session")
def gpu_device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _gather_where_jobs_have_to_share_launches(request, monkeypatch):
    """test_served_jobs_match_the_oracle wants at least two of its jobs in the
    pool together.  They arrive 0.5-5 ms apart and run for 0.5 ms each, so
    whether two meet is left to chance unless the server gathers them."""
    if request.node.name == "test_served_jobs_match_the_oracle":
        from paper_1107_4543_amd.serve import Server
        monkeypatch.setattr(Server, "__init__", functools.partialmethod(Server.__init__, gather_ms=2.0))
