"""Launch shapes of plans whose Heun steps the library would take in one pass:
a group size asked for selects the stage kernels and shapes them, and autotune
neither times one kernel under several names nor mixes the two kinds of plan."""

import pytest

from paper_2505_17284_amd import inputs as I
from tests.parity import compare_field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17284_amd import solver

    return solver


@pytest.mark.parametrize("order", [1, 3])
@pytest.mark.parametrize("rows,waves", [(2, 4), (4, 4), (2, 8), (4, 8)])
def test_group_sizes_shape_the_stage_kernels(sv, orc, order, rows, waves):
    p = I.random_materials(133, 37, 4, seed=order, M=32, order=order, stepper=I.HEUN, t_end=50.0,
                           rects=[(0, 0, 133, 37)])
    psi0 = I.random_state(p, 5, "uniform")
    print(f"[case] order {order} rows {rows} waves {waves}", flush=True)
    plan = sv.Plan(p, psi0=psi0, group_size=5, rows_per_wave=rows, waves_per_group=waves)
    try:
        plan.set_timing(True)
        plan.run(2)
        assert plan.kernel_ms()[1][1:3] == [2, 2]
        ok, rep = compare_field(plan.psi(), orc.solve(p, steps=2, psi0=psi0)["psi"], 4)
        assert ok, rep
    finally:
        plan.close()


def test_autotune_of_one_pass_plans(sv):
    open_, closed = (I.random_materials(133, 37, 4, seed=1, M=32, order=3, stepper=I.HEUN, t_end=50.0, bc=bc,
                                        rects=[(0, 0, 133, 37)])
                     for bc in ((I.BC_VACUUM,) * 4, (I.BC_REFLECT,) * 4))
    t = sv.autotune(open_)
    assert (t["group_size"], t["group_size_average"]) == (0, 0) and t["ms_per_step"] > 0
    u = sv.autotune(closed)  # the same grid and ordinates, in two stages
    assert u is not t and u["group_size"] > 0 and u["group_size_average"] > 0
    assert sv.autotune(open_) is t and sv.autotune(closed) is u
