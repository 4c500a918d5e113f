import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running test")


@pytest.fixture(scope="session")
def orc():
    import oracle
    oracle.build(force=False)
    return oracle


def qdict(names, values):
    return {n: float(v) for n, v in zip(names, values)}


# Tests that expect minmod (order 2) Heun steps of large FP32 plans in one pass
# over psi. They take the two stage kernels at every size (the rule in
# snrt_plan.cpp, with what it measured), so the launch counts that these tests
# ask for are wrong; test_gpu_minmod_routes.py has the same plans with the
# right ones.
_ONE_PASS_MINMOD = (
    ("test_gpu_heun_pass.py", "test_strip_band_and_ordinate_edges",
     lambda params: params.get("order") == 2),
    ("test_gpu_transfers.py", "test_static_area_without_room_for_more_than_two_stages", lambda params: True),
)


def pytest_collection_modifyitems(items):
    for item in items:
        call = getattr(item, "callspec", None)
        for path, name, when in _ONE_PASS_MINMOD:
            if item.path.name == path and getattr(item, "originalname", "") == name \
                    and when(call.params if call else {}):
                item.add_marker(pytest.mark.xfail(strict=True, raises=AssertionError,
                                                  reason="minmod Heun steps take two stages at every size"))
