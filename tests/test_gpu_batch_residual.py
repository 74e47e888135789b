"""rmrt_batch_residual (all domains in one launch) against rmrt_residual of the
same domains as contexts of their own, bit for bit: domains of one workgroup, of
many and of the most the reduction uses, periodic and walled ones in one batch,
solid nodes, natural and swapped layouts, a domain that starts again."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2206_00366_amd import rmrt
    return rmrt


def fields(p, k):
    N = p["n"][0] * p["n"][1] * p["n"][2]
    g = torch.Generator(device="cuda").manual_seed(k)
    d = 2 if p["lattice"] == "Q9" else 3
    rho = 1 + 1e-3 * torch.randn(N, generator=g, device="cuda", dtype=torch.float64)
    return rho, 1e-2 * torch.randn((d, N), generator=g, device="cuda", dtype=torch.float64)


@pytest.mark.parametrize("lattice,storage,pattern,sizes", [
    ("Q9", "f32dev", "AA", [(5, 3, 1), (300, 200, 1), (900, 700, 1)]),
    ("Q9", "f64", "AB", [(16, 16, 1), (257, 129, 1)]),
    ("Q27", "f32dev", "AA", [(16, 9, 7), (33, 40, 28)]),
    ("Q19", "f16dev", "AA", [(17, 12, 10), (64, 20, 20)]),
])
def test_batch_residual_matches_single_domains(R, lattice, storage, pattern, sizes):
    print(f"[batch residual] {lattice} {storage} {pattern}", file=sys.stderr, flush=True)
    ps, solids = [], []
    for k, n in enumerate(sizes):
        ps.append(dict(lattice=lattice, storage=storage, pattern=pattern, n=n, dx=(1.0, 0.5, 1.0), nu=0.1,
                       wall_faces=12 if k % 2 else 0))
        solids.append((np.random.default_rng(k).random(n[0] * n[1] * n[2]) < 0.05).astype(np.uint8))
    batch = R.Batch([R.make_params(**p) for p in ps], solids=solids)
    doms = []
    for k, p in enumerate(ps):
        rho, u = fields(p, k)
        batch.domains[k].set_fields(rho, u)
        doms.append(R.Domain(R.make_params(**p), rho, u, solid=solids[k]))
    for steps in (0, 2, 1, 4):
        batch.step(steps)
        for d in doms:
            d.step(steps)
        assert batch.residuals() == [d.residual() for d in doms], steps
    # one domain starts again: its next residual is +inf, the others go on
    rho, u = fields(ps[-1], 77)
    batch.domains[-1].set_fields(rho, u)
    r = batch.residuals()
    assert r[-1] == float("inf") and all(np.isfinite(v) for v in r[:-1])
    batch.close()
    for d in doms:
        d.close()
