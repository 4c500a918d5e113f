"""Rounding of the scalar flux of first-order Euler steps: small grids take groups
of as few as two ordinates, whose partials are summed in FP64. A partial of n
ordinates is rounded at most n times (each ordinate's fused multiply-add) and
phi once, each by at most 2^-24 of sum w |psi|: (n + 1) 2^-24 of that."""

import numpy as np
import pytest

from paper_2505_17284_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17284_amd import solver

    return solver


@pytest.mark.parametrize("n,M", [(70, 32), (104, 64), (133, 128)])
def test_phi_of_small_euler_steps(sv, n, M):
    p = I.lattice(n, M, order=1, stepper=I.EULER)
    psi0 = np.random.default_rng(n).uniform(0.2, 1.0, (M, n, n)).astype(np.float32)
    print(f"[case] {n} {M}", flush=True)
    plan = sv.Plan(p, psi0=psi0)
    try:
        plan.run(1)
        psi, phi, gs = plan.psi(), plan.phi().astype(np.float64), plan.info["group_size"]
    finally:
        plan.close()
    w, psi = p.quad.w.astype(np.float32).astype(np.float64), psi.astype(np.float64)
    exact, size = (np.einsum("k,kji->ji", w, a) for a in (psi, np.abs(psi)))
    worst = float(np.max(np.abs(phi - exact) / size))
    assert worst <= (gs + 1) * 2.0 ** -24, (worst, gs)
