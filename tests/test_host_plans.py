"""Bounds of the workspace layout and of every kernel's LDS plan, checked on the CPU: the index
helpers the kernels share with the host are compiled by hipcc into a small host
program (tests/host_plans.hip) that walks the extreme accepted shapes.  GPU sanitizers are not
available on the target machines; this is the net under the carved regions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "host_plans")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function",
                           "-Wno-unused-value", "-o", exe, os.path.join(ROOT, "tests", "host_plans.hip")])
    return exe


def test_workspace_and_lds_plans_stay_in_bounds(host_plans):
    run = subprocess.run([host_plans], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-2000:]
    assert "host plans ok" in run.stdout


def _pass_plans(host_plans, calls):
    """(waves, rounds) of k_logits_pass for (type, hidden rows, beams, V, d, pitch); (0, 0): another kernel's call."""
    text = "".join("%d %d %d %d %d %d\n" % ((2 if c[0] == "bf16" else 4,) + c[1:]) for c in calls)
    run = subprocess.run([host_plans, "pass"], input=text, capture_output=True, text=True, check=True)
    return [tuple(map(int, line.split())) for line in run.stdout.splitlines()]


def test_shapes_of_the_pass_tests_reach_it(host_plans):
    """The GPU tests of k_logits_pass name the split each shape has; more than 512 streamed tiles, so that no other plan is ahead of it."""
    import test_gpu_pass
    got = _pass_plans(host_plans, [(ty, S * B, B, V, d, ld) for ty, V, d, ld, S, B, _, _ in test_gpu_pass.SHAPES])
    assert got == [s[6:] for s in test_gpu_pass.SHAPES]
    assert all(V > 512 * 16 and S * B <= (16 if ty == "bf16" else 48) for ty, V, _, _, S, B, _, _ in test_gpu_pass.SHAPES)
    assert {g[0] for g in got} == set(range(4, 13)) and {g[1] for g in got} == set(range(1, 6))


def test_extreme_values_reach_both_kernels_for_a_few_rows(host_plans):
    import test_gpu_extreme_values as t
    calls = [(n, (ty, S * B, B, V, d, d)) for n, (S, B, V, _, _, ds, tys) in t._DRIVERS.items() if n.startswith(("few", "pass"))
             for d in ds for ty in tys]
    for (name, _), plan in zip(calls, _pass_plans(host_plans, [c for _, c in calls])):
        assert (plan[0] > 0) == name.startswith("pass"), (name, plan)


def test_every_trace_point_has_its_place():
    """A build with phase timestamps: every point of every kernel writes inside the arrays (a static_assert in the macros)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    run = subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only", "-std=c++17", "-w", "-DLSHBEAM_TRACE",
                          os.path.join(ROOT, "paper_1806_00588_amd", "csrc", "lshbeam.hip")], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-3000:]
