"""FP64 domains on passes of several steps (k_tile_steps, k_two_step) and rD2Q9
domains kept on single steps, run by tests/test_gpu_checked_passes.py in a child
process, once with the production library and once with the index-checked one
(RMRT_LIBRARY).

Usage: python tests/checked_pass_cases.py OUT.npz
Writes every case's densities to OUT.npz and prints a line per case: the neighbour
indices found out of range (-1 in the production build), the launches of the last
call and whether the populations are those of single steps."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.join(ROOT, "tests"))

import numpy as np  # noqa: E402
import torch  # noqa: E402

from gpu_util import WALLS, circle_mask  # noqa: E402
from paper_2206_00366_amd import rmrt as R  # noqa: E402


def violations(dom):
    return dom.checked_violations() if R.checked_build() else -1


def make(prm, solid, single):
    n = prm["n"]
    N = n[0] * n[1] * n[2]
    rng = np.random.default_rng(N)
    rho = 1.0 + 1e-3 * rng.uniform(-1, 1, N)
    u = 0.02 * rng.uniform(-1, 1, (2 if n[2] == 1 else 3, N)) if prm.get("equation", "NSE") == "NSE" else None
    dom = R.Domain(R.make_params(**prm, storage="f64"), rho, u, solid=None if solid is None else solid.astype(np.uint8))
    if single:
        dom.set_launch(*dom.get_launch())
    return dom


Q9 = dict(lattice="Q9", dx=(1.0, 0.5, 1.0), nu=0.05)
NCDE = dict(lattice="Q9", equation="NCDE", dx=(1.0, 0.5, 1.0), D0=0.01, D2=1.0, adv=(0.05, 0.02, 0.0), rho0=0.0)
Q19 = dict(lattice="Q19", dx=(1.0, 1.0, 2.0), nu=0.05)
CASES = [  # name, parameters, solid mask
    ("q9_solid_aa", dict(Q9, n=(40, 21, 1), wall_faces=WALLS["y"], pattern="AA"), circle_mask((40, 21, 1), (12, 10), 4)),
    ("q9_solid_ab", dict(Q9, n=(40, 21, 1), pattern="AB"), circle_mask((40, 21, 1), (20, 10), 5)),
    ("q9_walls_tiles", dict(Q9, n=(700, 90, 1), wall_faces=15, pattern="AA"), None),
    ("q9_periodic_smallest", dict(Q9, n=(8, 8, 1), pattern="AB"), None),
    ("q9_ncde", dict(NCDE, n=(333, 217, 1), pattern="AA"), None),
    ("q19_whole_rows_aa", dict(Q19, n=(96, 96, 96), pattern="AA"), None),
    ("q19_split_rows_ab", dict(Q19, n=(341, 90, 80), pattern="AB"), None),
]


def main(out_path):
    out = {}
    for name, prm, solid in CASES:
        dom, ref = make(prm, solid, False), make(prm, solid, True)
        for steps in (8, 1, 11):
            dom.step(steps)
            ref.step(steps)
        same = torch.equal(dom.populations(), ref.populations())
        out[name] = dom.moments()[0].cpu().numpy()
        print("case", name, violations(dom), violations(ref), dom.step_launches(8), ref.step_launches(8), int(same),
              flush=True)
        dom.close()
        ref.close()
    np.savez(out_path, **out)
    if R.checked_build():
        # the checks themselves, with the bound lowered below the node count (every
        # access stays inside the buffers)
        for name, prm, solid in (CASES[2], CASES[5]):
            dom = make(prm, solid, False)
            dom.step(8)
            clean = dom.checked_violations()
            dom.checked_set_limit(dom.N - 300)
            dom.step(8)
            print("selftest", name, clean, dom.checked_violations(), flush=True)
            dom.close()


if __name__ == "__main__":
    main(sys.argv[1])
