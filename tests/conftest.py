import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (runs the HIP library)")
    config.addinivalue_line("markers", "slow: longer CPU test")


@pytest.fixture(scope="session", autouse=True)
def _oracle_threads():
    from oracle import pyoracle
    pyoracle.set_threads(min(16, os.cpu_count() or 1))
    yield


@pytest.fixture(autouse=True)
def _seeded_draws(request):
    """GPU tests that draw without a generator of their own draw the same each run"""
    if request.node.get_closest_marker("gpu"):
        import torch

        torch.manual_seed(0)
    yield
