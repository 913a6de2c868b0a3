import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle_mod():
    import oracle
    oracle.build()
    return oracle


@pytest.fixture(autouse=True)
def no_handles_left_to_collect(request):
    """A handle that an earlier test left in a cycle (an exception that pytest.raises holds, with its frames) is destroyed when the
    cycle is collected, which frees device memory; inside a graph's capture that would end the capture."""
    if "graph" in request.node.name:
        gc.collect()
