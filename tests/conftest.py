import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run through the C-ABI HIP library)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle

    _oracle.build()
    return _oracle


@pytest.fixture(autouse=True, scope="module")
def _no_garbage_left_for_the_next_module():
    """Tensors that a test left in reference cycles (tracebacks) are freed here and not at some allocation of a later
    test that watches the allocator."""
    yield
    gc.collect()
