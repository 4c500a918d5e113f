"""The one-pass Heun step where the last strip of 112 columns is one to three
columns wide: the halo of the strip before it then holds the grid's last columns
and its ghost cells, whose rules it has to apply too. Against the oracle with the
tolerances of tests/parity.py."""

import numpy as np
import pytest

from paper_2505_17284_amd import inputs as I
from tests.parity import compare_field

pytestmark = pytest.mark.gpu

INFLOW = ((I.BC_INFLOW,) * 4, (0.5, 0.8, 1.0, 0.25))


@pytest.fixture(scope="module")
def sv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17284_amd import solver

    return solver


@pytest.mark.parametrize("order", [1, 3])
@pytest.mark.parametrize("nx", [225, 226, 227, 337, 338])
def test_narrow_last_strips(sv, orc, nx, order):
    p = I.random_materials(nx, 21, 4, seed=nx, M=32, order=order, stepper=I.HEUN, bc=INFLOW[0], inflow=INFLOW[1],
                           t_end=50.0, rects=[(0, 0, nx, 21)])
    psi0 = I.random_state(p, nx, "uniform")
    print(f"[case] {nx} order {order}", flush=True)
    plan = sv.Plan(p, psi0=psi0)
    try:
        plan.set_timing(True)
        plan.run(3)
        assert plan.kernel_ms()[1][1] == 0
        psi = plan.psi()
    finally:
        plan.close()
    ok, rep = compare_field(psi, orc.solve(p, steps=3, psi0=psi0)["psi"], 6)
    assert ok, rep
