import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=[0, 2], ids=["auto", "blocks"])
def both_paths(request):
    """16-bit data at head_dim 64 / 128: once as the library chooses, which for short sequences on few chains is the launch that looks
    back over all positions, and once on the block recurrence's kernels.  (Resetting is the test file's own fixture's part.)"""
    from paper_2401_04658_amd import binding
    binding.la2_set_scan_variant(request.param)
    return request.param
