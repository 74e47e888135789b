"""The rules that choose passes of several steps (csrc/sweep_plan.hpp), compiled for
the CPU: a call is split into pairs of passes of lengths that pay, and measured
losses are not taken."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_take_what_pays(tmp_path):
    exe = str(tmp_path / "rule")
    src = os.path.join(ROOT, "tests", "sweep_plan", "rule.cpp")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", src, "-o", exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok"), (res.stdout, res.stderr[-3000:])
