"""Launch sequences of the library, on the CPU: every test body runs in a
process of its own on a HIP runtime that only records (host_launches.Host)."""

import inspect
import json
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def workdir(tmp_path_factory):
    return str(tmp_path_factory.mktemp("hip_stub"))


def _on_host(workdir, body, *args):
    """body(host, *args) in another process; its value (JSON)."""
    code = ("import json, sys\nfrom tests.host_launches import Host\nfrom paper_2505_17284_amd import inputs as I\n"
            + textwrap.dedent(inspect.getsource(body))
            + f"\nprint('\\n@' + json.dumps({body.__name__}(Host({workdir!r}), *json.loads({json.dumps(args)!r}))))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.rsplit("\n@", 1)[1])


def _kernels_of_steps(host, kind, n, M, order, stepper, steps):
    p = getattr(I, kind)(n, M, order=order, stepper=stepper)  # noqa: F821
    h = host.plan(p)
    host.launches()
    host.L.check(host.lib.sn_plan_run(h, steps, None), "run")
    return [k for k, _, _ in host.launches()]


TWO_STAGES = ["sn_stage_kernel", "sn_qoi_finalize_kernel"] * 2


@pytest.mark.parametrize("kind,n,M", [("lattice", 70, 32), ("lattice", 280, 256), ("lattice", 700, 256),
                                      ("cavity", 437, 128), ("cavity", 1300, 512), ("hohlraum", 390, 256)])
def test_minmod_heun_steps_are_two_stages_at_every_size(workdir, kind, n, M):
    """Minmod amplifies a change of rounding without end, so that its steps are
    the same two launches whatever the size."""
    assert _on_host(workdir, _kernels_of_steps, kind, n, M, 2, 1, 3) == TWO_STAGES * 3


@pytest.mark.parametrize("order", [1, 3])
def test_heun_steps_of_orders_1_and_3_are_one_pass(workdir, order):
    got = _on_host(workdir, _kernels_of_steps, "lattice", 70, 32, order, 1, 2)
    assert got == ["sn_heun_kernel", "sn_heun_finalize_kernel"] * 2 + ["sn_materialize_kernel"]


@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("n,M", [(70, 32), (104, 64), (140, 64), (200, 64), (208, 64), (280, 128), (333, 128), (560, 256)])
def test_euler_groups_of_limited_orders_are_those_of_the_update_stage(n, M, order):
    """The grouping decides how phi is rounded, and the limited orders amplify
    that: Euler keeps the groups of Heun's update stage there."""
    from paper_2505_17284_amd import inputs as I
    from paper_2505_17284_amd import solver

    a, b = (solver.plan_info(I.lattice(n, M, order=order, stepper=s)) for s in (I.EULER, I.HEUN))
    assert a["group_size"] == b["group_size"]


def _threads_of_init(host, nx, M, order, stepper):
    quad = I.tessellation_quadrature(22) if M == 1936 else None  # noqa: F821
    p = I.lattice(nx, 32 if quad else M, order=order, stepper=stepper, quad=quad)  # noqa: F821
    h = host.plan(p, bind=False)
    host.L.check(host.bind(h), "bind")
    host.launches()
    host.L.check(host.lib.sn_plan_init(h, *host.addresses(4 * p.M * p.ny * p.nx), None), "init")
    host.L.check(host.lib.sn_plan_run(h, 1, None), "run")
    return [p.M * p.ny * p.nx, host.launches()]


@pytest.mark.parametrize("nx,M,order,stepper", [(700, 256, 2, 1), (1500, 1936, 1, 0), (1500, 1936, 3, 1)])
def test_launches_of_large_states_stay_below_2_32_threads(workdir, nx, M, order, stepper):
    """HIP takes fewer than 2^32 threads per launch; 1500^2 x 1936 has 4.4e9
    cell-ordinates, and psi0 is unpacked a thread each."""
    n, launches = _on_host(workdir, _threads_of_init, nx, M, order, stepper)
    assert all(blocks * threads < 2 ** 32 for _, blocks, threads in launches), launches
    unpacked = [blocks * threads for k, blocks, threads in launches if k == "sn_pack_kernel"]
    assert n <= sum(unpacked) < n + 256 * len(unpacked) and len(unpacked) <= 1 + n // 2 ** 31
