import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (runs the HIP library through the C ABI)")


def read_golden(name):
    """Parses a tests/golden/*.txt fixture: '# comment' lines, 'key: v v v' records."""
    out = {}
    with open(os.path.join(ROOT, "tests", "golden", name)) as f:
        for line in f:
            line = line.split("#", 1)[0].strip()
            if not line:
                continue
            key, vals = line.split(":", 1)
            out[key.strip()] = [float(v) for v in vals.split()]
    return out


@pytest.fixture(scope="session")
def golden():
    return read_golden


@pytest.fixture(autouse=True, scope="module")
def _no_garbage_of_other_modules():
    """Device memory that earlier tests' reference cycles still hold is freed here and not at some later allocation, between
    two readings of torch's memory statistics for instance."""
    gc.collect()
    yield
