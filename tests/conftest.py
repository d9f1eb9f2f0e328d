import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


def pytest_runtest_setup(item):
    """A GPU test that is run fails where there is no GPU, also if its own fixture
    would skip it: a broken machine must not pass for a tested one."""
    if item.get_closest_marker("gpu"):
        import torch
        if not torch.cuda.is_available():
            pytest.fail("GPU tests need a GPU")
