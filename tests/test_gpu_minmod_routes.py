"""Minmod Heun steps take the two stage kernels at every size: the plans of
test_gpu_heun_pass.py's large order-2 cases and the 700^2 x 256 lattice, against
the oracle with the tolerances of tests/parity.py, and in the static area
against caller scratch bit for bit."""

import numpy as np
import pytest

from paper_2505_17284_amd import inputs as I
from tests.parity import compare_field, compare_qoi

pytestmark = pytest.mark.gpu

INFLOW = ((I.BC_INFLOW, I.BC_VACUUM, I.BC_INFLOW, I.BC_INFLOW), (0.5, 0.0, 1.0, 0.25))


@pytest.fixture(scope="module")
def sv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_17284_amd import solver

    return solver


def _run(sv, p, steps, psi0=None, **kw):
    plan = sv.Plan(p, psi0=psi0, **kw)
    try:
        plan.set_timing(True)
        plan.run(steps)
        counts = plan.kernel_ms()[1]
        return dict(plan.qoi(), psi=plan.psi(), phi=plan.phi()), counts
    finally:
        plan.close()


@pytest.mark.parametrize("nx,ny,quad", [(8, 776, "T22"), (111, 56, "T22"), (120, 53, "T22"), (337, 19, "T22"),
                                        (225, 106, 512)])
def test_large_minmod_plans_against_the_oracle(sv, orc, nx, ny, quad):
    p = I.random_materials(nx, ny, 4, seed=100 * nx + ny, M=quad if isinstance(quad, int) else 32, order=2,
                           stepper=I.HEUN, bc=INFLOW[0], inflow=INFLOW[1], t_end=50.0, rects=[(0, 0, nx, ny)])
    if not isinstance(quad, int):
        p = p.replace(quad=I.tessellation_quadrature(int(quad[1:])))
    psi0 = I.random_state(p, nx + ny, "smooth")
    print(f"[case] {p.name} M={p.M}", flush=True)
    g, counts = _run(sv, p, 3, psi0)
    assert counts[1] == 3 and counts[2] == 3, counts
    o = orc.solve(p, steps=3, psi0=psi0)
    ok, rep = compare_qoi(g["qoi"], g["qoi_int"], dict(zip(o["names"], o["qoi"])), dict(zip(o["names"], o["qoi_int"])))
    assert ok, rep
    for name in ("psi", "phi"):
        ok, rep = compare_field(g[name], o[name], 6)
        assert ok, f"{name}: {rep}"


def test_the_static_area_gives_the_bits_of_caller_scratch(sv):
    p = I.lattice(700, 256, order=2, stepper=I.HEUN)
    out = []
    for static in (True, False):
        print(f"[case] static {static}", flush=True)
        g, counts = _run(sv, p, 4, static_scratch=static)
        assert counts[1] == 4 and counts[2] == 4, counts
        out.append(g)
    for k in ("psi", "phi"):
        assert np.array_equal(out[0][k], out[1][k]), k
    assert out[0]["qoi"] == out[1]["qoi"] and out[0]["qoi_int"] == out[1]["qoi_int"]
