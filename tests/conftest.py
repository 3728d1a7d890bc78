import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=["one_launch", "several_launches"])
def launches(request, monkeypatch):
    """Predicted calls of small layouts as they come, in one launch, and by the kernels that larger layouts take (a stream
    launch shape that is set keeps contexts to those; 1 is the shape that they have anyway)."""
    if request.param == "several_launches":
        monkeypatch.setenv("DGS_STREAM_QUADS", "1")
    return request.param


@pytest.fixture(scope="session")
def oracle():
    from oracle import dgs_oracle
    dgs_oracle.build()
    return dgs_oracle
