import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    # GPU tests are only meaningful on a GPU machine; without one they are skipped, not failed.
    try:
        import torch
        has_gpu = torch.cuda.is_available()
    except Exception:  # pragma: no cover
        has_gpu = False
    if has_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for it in items:
        if "gpu" in it.keywords:
            it.add_marker(skip)


@pytest.fixture
def no_automatic_collection():
    """For tests that capture graphs.  A graph that is left in a reference cycle (by exception info and its frame) is destroyed by
    whatever garbage collection comes next; if that starts inside a capture, the destructor's synchronisation, which a capture
    forbids, ends the process."""
    gc.collect()
    gc.disable()
    try:
        yield
    finally:
        gc.enable()
