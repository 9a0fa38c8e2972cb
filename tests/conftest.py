import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def per_launch():
    """Tensors that a launch of the batched calls holds (more than the *_batch_capacity() calls promise)."""
    with open(os.path.join(ROOT, "paper_2510_11400_amd", "csrc", "fh_batch.hpp")) as f:
        return int(re.search(r"constexpr int kBatch = (\d+);", f.read()).group(1))


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")
