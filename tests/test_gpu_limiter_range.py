"""Order 3 at the ends of FP32's range, where the limiter's b^2 or its
regularisation h^12 is infinite: a direction without a gradient leaves the
limiter at 1 there, and the state finite."""

import numpy as np
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


@pytest.mark.parametrize("stepper", [I.EULER, I.HEUN])
def test_steep_beam_without_a_gradient_along_y(sv, stepper):
    """Differences between neighbours above 2^64, uniform along y."""
    g = 1e21
    p = I.beam(nx=24, ny=3, g=g, order=3, stepper=stepper)
    print(f"[case] beam {stepper}", flush=True)
    psi = sv.solve(p, steps=8, return_psi=True)["psi"]
    assert np.isfinite(psi).all()
    steps = np.diff(psi.astype(np.float64), axis=2)
    assert (np.abs(steps) > 2.0 ** 64).any()  # b^2 overflows
    assert np.array_equal(psi, np.broadcast_to(psi[:, :1], psi.shape))


@pytest.mark.parametrize("stepper", [I.EULER, I.HEUN])
def test_uniform_medium_of_huge_cells(sv, orc, stepper):
    """h^12 above the largest float; an infinite medium stays uniform."""
    p = I.homogeneous(nx=6, ny=5, sigma_a=7e-5, sigma_s=4e-5, q=1.3e-4, order=3, stepper=stepper, h=2000.0, t_end=6000.0)
    print(f"[case] huge cells {stepper}", flush=True)
    g, o = sv.solve(p, return_psi=True), orc.solve(p)
    ok, rep = compare_field(g["psi"], o["psi"], 2 * p.M)
    assert ok, rep
