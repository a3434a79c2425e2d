import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    import torch
    if torch.cuda.is_available():
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture
def tuning():
    """lava.set_tuning for the duration of one test (launch shapes chosen through the C ABI); the
    library's own choices are restored afterwards."""
    from paper_2509_09754_amd import lava
    yield lava.set_tuning
    lava.set_tuning()


@pytest.fixture
def launches():
    """launches(call): what the call returns, and how often it launched each kernel of the library."""
    import torch
    from paper_2509_09754_amd import lava

    def count(call):
        lava.prof_enable(True), lava.prof_reset()
        try:
            out = call()
            torch.cuda.synchronize()
            return out, {name: n for name, (_, n) in lava.prof_read().items()}
        finally:
            lava.prof_enable(False), lava.prof_reset()
    return count
