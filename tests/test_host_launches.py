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
    """Minmod amplifies a change of rounding to per cents of a value, so that its
    steps are the same two launches whatever the size."""
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


@pytest.mark.parametrize("nx,M,order,stepper", [(7, 32, 2, 1), (700, 256, 2, 1), (1500, 1936, 1, 0), (1500, 1936, 3, 1)])
def test_launches_of_large_states_stay_below_2_32_threads(workdir, nx, M, order, stepper):
    """HIP takes fewer than 2^32 threads per launch; 1500^2 x 1936 has 4.4e9
    cell-ordinates, and psi0 is unpacked a thread each."""
    n, launches = _on_host(workdir, _threads_of_init, nx, M, order, stepper)
    assert all(blocks * threads < 2 ** 32 for _, blocks, threads in launches), launches
    unpacked = [blocks * threads for k, blocks, threads in launches if k == "sn_pack_kernel"]
    assert n <= sum(unpacked) < n + 256 * len(unpacked) and len(unpacked) <= 1 + n // 2 ** 31


def _launches_of_one_cell(host, nx, ny):
    p = I.random_materials(nx, ny, 1, seed=1, M=32, order=1, rects=[])  # noqa: F821
    h = host.plan(p, bind=False)
    host.L.check(host.bind(h), "bind")
    host.launches()
    host.L.check(host.lib.sn_plan_init(h, *host.addresses(4 * p.M * nx * ny), None), "init")
    return host.launches()


@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (1, 3)])
def test_psi0_of_the_smallest_grids_is_unpacked_once(workdir, nx, ny):
    unpacked = [b * t for k, b, t in _on_host(workdir, _launches_of_one_cell, nx, ny) if k == "sn_pack_kernel"]
    assert unpacked == [256]


def _reads_after_a_failed_run(host, order, graph, function, k):
    p = I.lattice(70, 32, order=order, stepper=I.HEUN)  # noqa: F821
    h = host.plan(p)
    if graph:
        host.L.check(host.lib.sn_plan_use_graph(h, graph), "graph")
    host.launches()
    host.fail(function, k)
    out = dict(run=host.lib.sn_plan_run(h, 7, None), replays=host.stub.stub_graph_replays())
    host.launches()
    psi, q = host.addresses(1 << 26)[0], host.L.SnQoi()

    def reads():
        import numpy as np
        a = np.zeros((p.M, p.ny, p.nx), np.float32)
        st = host.lib.sn_plan_qoi(h, host.L.ctypes.byref(q), None)
        return [host.lib.sn_plan_read_psi(h, a.ctypes.data, None), host.L.SN_OK if st == host.L.SN_ERR_NONFINITE else st]

    out["reads"] = reads()
    host.fail("", 0)
    out["settle"] = host.lib.sn_plan_run(h, 0, None)
    out["launches_then"] = [n for n, _, _ in host.launches()]
    out["reads_then"] = reads()
    return out


@pytest.mark.parametrize("graph,function,k", [(0, "hipLaunchKernel", k) for k in (1, 2, 3, 4, 9, 14, 15)]
                         + [(2, "hipGraphInstantiate", 1), (2, "hipGraphInstantiate", 2), (2, "hipGraphLaunch", 1),
                            (2, "hipGraphLaunch", 3), (2, "hipStreamEndCapture", 2)])
def test_a_run_that_fails_between_one_pass_steps_is_not_read_as_if_it_had_ended(workdir, graph, function, k):
    """After a step the buffer lacks the step's shift until the run's end adds
    it: a run that ends before has SN_ERR_STATE for readers until the state is
    settled (any run, also of no steps, does)."""
    r = _on_host(workdir, _reads_after_a_failed_run, 3, graph, function, k)
    assert r["run"] == 3  # SN_ERR_DEVICE
    steps = (k - 1) // 2 if not graph else r["replays"]
    ok, state = 0, 7
    assert r["reads"] == ([state, state] if steps > 0 else [ok, ok])
    assert r["settle"] == ok and r["reads_then"] == [ok, ok]
    assert r["launches_then"].count("sn_materialize_kernel") == (1 if steps > 0 else 0)


def _kernels_of_shaped_steps(host, order, shape):
    h = host.plan(I.lattice(140, 64, order=order, stepper=I.HEUN), **shape)  # noqa: F821
    host.launches()
    host.L.check(host.lib.sn_plan_run(h, 2, None), "run")
    return [k for k, _, _ in host.launches()]


@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("shape", [dict(group_size=8), dict(group_size_average=16), dict(group_size=5, rows=4, waves=8)])
def test_ordinate_groups_asked_for_shape_the_steps(workdir, order, shape):
    assert _on_host(workdir, _kernels_of_shaped_steps, order, shape) == TWO_STAGES * 2


@pytest.mark.parametrize("order", [1, 3])
def test_rows_and_waves_alone_leave_the_choice(workdir, order):
    """Batches name them for every member, whose steps are those of the plan alone."""
    got = _on_host(workdir, _kernels_of_shaped_steps, order, dict(rows=2, waves=4))
    assert got[:2] == ["sn_heun_kernel", "sn_heun_finalize_kernel"]


def _bound_twice(host):
    p = I.lattice(700, 256, order=3, stepper=I.HEUN)  # noqa: F821
    h = host.plan(p, bind=False)
    out, phi = [], host.addresses(1 << 23)[0]
    info = host.info(h)
    for static in (False, True, False):
        bind = (host.lib.sn_plan_bind_static(h, *host.addresses(info["psi_bytes"], info["psi_bytes"])) if static
                else host.bind(h))
        host.L.check(bind, "bind")
        host.L.check(host.lib.sn_plan_init(h, None, None), "init")
        host.launches()
        host.L.check(host.lib.sn_plan_run(h, 2, None), "run")
        host.L.check(host.lib.sn_plan_read_phi(h, phi, None), "phi")
        out.append([host.info(h)["scratch_bytes"], [k for k, _, _ in host.launches()]])
    return out


def test_a_plan_bound_to_the_static_area_and_then_to_caller_scratch(workdir):
    """The static area holds this plan only without the one-pass areas and the
    packed plane; scratch of the size sn_plan_get_info asks for has them again."""
    first, static, then = _on_host(workdir, _bound_twice)
    assert first[0] > 64 << 20 and static[0] == then[0] == first[0]
    assert static[1] == TWO_STAGES * 2
    assert then[1] == first[1] == ["sn_heun_kernel", "sn_heun_finalize_kernel"] * 2 + ["sn_materialize_kernel",
                                                                                        "sn_pack_kernel"]


def _one_pass_launch(host, n, M, order):
    h = host.plan(I.lattice(n, M, order=order, stepper=I.HEUN))  # noqa: F821
    host.launches()
    host.L.check(host.lib.sn_plan_run(h, 1, None), "run")
    lds = host.lds()[0]
    return [*host.launches()[0], lds]


@pytest.mark.parametrize("n,M", [(1300, 32), (700, 32), (437, 32), (1300, 64), (560, 256)])
def test_the_last_round_of_one_pass_workgroups_is_not_nearly_empty(workdir, n, M):
    """Bands are cut for the workgroups that a compute unit holds, by waves (16)
    and by LDS (160 KiB)."""
    kernel, blocks, threads, lds = _on_host(workdir, _one_pass_launch, n, M, 3)
    assert kernel == "sn_heun_kernel"
    rounds = blocks / (256 * min(1024 // threads, 160 * 1024 // lds))
    assert rounds % 1 == 0 or rounds % 1 >= 0.4 or rounds > 4, rounds
