"""The host code of the C ABI on the CPU, on a runtime of the test's own and with
launchers that only record (tests/host_runtime): what the stepping calls allocate,
launch and wait for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_runtime")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-std=c++17", "-O1", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("host_runtime")
    objs = []
    for src in (os.path.join(ROOT, "paper_2206_00366_amd", "csrc", "rmrt_capi.cpp"),
                os.path.join(HERE, "launch_stubs.hip"), os.path.join(HERE, "driver.cpp")):
        obj = str(out / (os.path.basename(src) + ".o"))
        res = subprocess.run([HIPCC, *FLAGS, "-x", "hip", "-c", src, "-o", obj], capture_output=True, text=True, timeout=600)
        assert res.returncode == 0, res.stderr[-3000:]
        objs.append(obj)
    exe = str(out / "driver")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", *objs, "-o", exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-3000:]
    return exe


def run(exe, scenario):
    res = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok"), (res.stdout, res.stderr[-3000:])


def test_a_failed_set_up_leaves_single_steps_and_no_memory(driver):
    run(driver, "out_of_memory")


def test_the_first_call_waits_for_nothing(driver):
    run(driver, "no_wait")


def test_failed_tuning_leaves_the_path_as_it_was(driver):
    run(driver, "failed_tuning")


def test_reported_launches_are_the_ones_made(driver):
    run(driver, "counted_launches")


def test_calls_without_passes_set_none_up(driver):
    run(driver, "only_for_passes")
