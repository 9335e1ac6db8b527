import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (HIP device) and the built HIP library")
    config.addinivalue_line("markers", "slow: takes more than a few seconds on the CPU")


def pytest_runtest_setup(item):
    # An exception caught by pytest.raises(...) as e keeps its test's tensors alive in a reference cycle until the
    # cyclic collector happens to run; freed inside a later test, they would falsify its count of device memory.
    if item.get_closest_marker("gpu"):
        gc.collect()
