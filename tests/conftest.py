import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


# Tests that hold a value which was wrong.  They stay as they are and run; each
# is expected to fail, for the reason given.
WRONG_VALUES = {
    "test_gpu_foldin_runtime.py::test_refused_on_an_older_runtime":
        "fold-in serves on older HIP runtimes again: the fault there was unwritten padding of the drawn factors "
        "(test_gpu_foldin_padding.py, test_gpu_foldin_torch.py)",
}
for k in (65, 80, 81, 96, 100, 112, 113, 128):
    WRONG_VALUES["test_gpu_lowrank_wide.py::test_lowrank_above_64[97-%d]" % k] = (
        "97 rows above K = 64 take the blocked kernel again, 1.2 to 1.6 times as fast there as the rank-one path "
        "(test_gpu_lowrank_rule.py)")


def pytest_collection_modifyitems(items):
    for item in items:
        for name, why in WRONG_VALUES.items():
            if item.nodeid.endswith(name):
                item.add_marker(pytest.mark.xfail(strict=True, reason=why))


@pytest.fixture(scope="session")
def orc():
    import oracle

    oracle.build()
    return oracle
