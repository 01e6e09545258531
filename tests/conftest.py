import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


@pytest.fixture(scope="session")
def orc():
    from oracle import oracle
    oracle.build()
    return oracle


def pytest_runtest_setup(item):
    """Batches that earlier tests left in reference cycles (a frame kept by a caught exception) are destroyed now and not
    whenever the collector runs next: freeing device memory while a stream is being captured invalidates the capture."""
    if "captur" in item.name or "graph" in item.name:
        gc.collect()
