import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (runs through the HIP library)")
    config.addinivalue_line("markers", "slow: longer CPU test")


@pytest.fixture(autouse=True)
def default_kernels():
    """Whatever a test leaves in the process-wide kernel-family switch (an assertion may come before
    its reset), the next one starts with the automatic choice."""
    yield
    mod = sys.modules.get("paper_2609_16478_amd")
    if mod is not None:
        mod.set_dst_variant(0)
