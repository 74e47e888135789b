"""The work split of the two-step kernel (csrc/sweep_plan.hpp), compiled for the
CPU: items cover every node of a domain exactly once and fit their workgroup,
over sizes below, at and beyond the patch widths, whole rows and split ones."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_items_cover_the_domain_once(tmp_path):
    exe = str(tmp_path / "check")
    src = os.path.join(ROOT, "tests", "sweep_plan", "check.cpp")
    res = subprocess.run(["g++", "-std=c++17", "-O2", src, "-o", exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok"), (res.stdout, res.stderr[-3000:])
