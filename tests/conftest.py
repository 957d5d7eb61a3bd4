import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: takes more than a few seconds on the CPU")


def pytest_runtest_setup(item):
    # This test compares torch's allocated memory before and after its calls.  Tensors
    # of earlier tests that only a raised error's traceback still holds (a reference
    # cycle) would be freed whenever the collector happens to run, in between too.
    if item.name == "test_device_memory_unchanged":
        gc.collect()


@pytest.fixture(scope="session")
def c_oracle():
    import oracle
    if not oracle.c_oracle_available():
        from oracle import build as ob
        ob.build()
    return oracle
