import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="module", autouse=True)
def _no_garbage_of_other_modules():
    # tracebacks kept by pytest.raises hold the failed call's tensors in reference cycles; collected in the middle of a
    # later module, they change the allocator's counts that test_zz_no_alloc.py compares
    gc.collect()


@pytest.fixture(scope="session")
def orc():
    import oracle

    oracle.build()
    return oracle
