"""The index-checked build on passes of several steps in 2D and 3D and on the single
steps of the same domains (tests/checked_pass_cases.py): no neighbour index out of
range, the populations of single steps bit for bit, the production library's
densities; with the bound lowered the checks of both pass kernels count."""
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2206_00366_amd")


def _run(lib, out):
    res = subprocess.run([sys.executable, os.path.join(ROOT, "tests", "checked_pass_cases.py"), out],
                         env=dict(os.environ, RMRT_LIBRARY=lib), capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, res.stderr[-3000:]
    print(res.stdout, flush=True)
    return [ln.split() for ln in res.stdout.splitlines()]


def test_passes_find_no_index_out_of_range(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    checked = os.path.join(PKG, "librmrt_checked.so")
    assert os.path.exists(checked), "librmrt_checked.so is not built"
    prod_out, chk_out = str(tmp_path / "prod.npz"), str(tmp_path / "checked.npz")
    prod, chk = _run(os.path.join(PKG, "librmrt.so"), prod_out), _run(checked, chk_out)
    for lines, count in ((prod, "-1"), (chk, "0")):
        cases = [ln[1:] for ln in lines if ln and ln[0] == "case"]
        assert len(cases) == 7
        for name, dom, ref, passes, single, same in cases:
            assert dom == ref == count, (name, dom, ref)
            assert int(passes) < 8 and int(single) == 8, (name, passes, single)
            assert same == "1", name
    a, b = np.load(prod_out), np.load(chk_out)
    assert sorted(a.files) == sorted(b.files)
    for k in a.files:
        # the inserted checks may change which multiply-adds the compiler fuses: rounding of 20 steps
        fin = np.isfinite(a[k])
        assert np.array_equal(fin, np.isfinite(b[k])), k
        assert np.abs(a[k][fin] - b[k][fin]).max() <= 1e-13 * np.abs(a[k][fin]).max(), k
    tests = [ln for ln in chk if ln and ln[0] == "selftest"]
    assert len(tests) == 2
    for _, name, clean, lowered in tests:
        assert int(clean) == 0 and int(lowered) > 0, name
