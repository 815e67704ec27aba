import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.fixture(autouse=True)
def settings_as_they_start(request):
    """Every GPU test leaves the library's settings as a new process has them."""
    yield
    r = sys.modules.get("paper_1908_02518_amd")
    if r is None or request.node.get_closest_marker("gpu") is None:
        return
    r.set_shortcuts()
    r.set_reduced_storage()
    r.set_reduce_workgroups(0)
    r.batched_set_config()
    r.batched_set_spread()
    r.set_working_column()  # and both sweeps
