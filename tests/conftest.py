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
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")


@pytest.fixture(scope="module", autouse=True)
def nothing_left_over():
    """Device memory that earlier modules' reference cycles still hold (a caught exception and its frames) is given back
    before a module starts, not in the middle of a test that counts allocations."""
    gc.collect()
    yield
