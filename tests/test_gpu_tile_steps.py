"""Several steps per pass on rD2Q9 (k_tile_steps) against single steps of the same
library: the same collision with the same roundings, so the populations agree
bit for bit; the single steps are compared with the oracle elsewhere.
rmrt_set_launch / rmrt_batch_set_config keep a domain or a batch on single steps."""
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


def params(kind, n, storage, pattern):
    p = dict(lattice="Q9", n=(*n, 1), storage=storage, pattern=pattern, dx=(1.0, 0.5, 1.0), nu=0.05, rho0=1.0)
    solid = None
    if kind == "walls":
        p.update(wall_faces=15, force=(1e-4, 2e-5, 0.0) if storage == "f32dev" else (0.0, 0.0, 0.0))
    if kind == "solid":
        p.update(wall_faces=3)
        solid = (np.random.default_rng(n[0]).random(n[0] * n[1]) < 0.1).astype(np.uint8)
    if kind == "ncde":
        p.update(equation="NCDE", D0=0.05, D2=0.5, adv=(0.02, 0.01, 0.0), rho0=0.5,
                 source=1e-4 if storage == "f32dev" else 0.0)
    return p, solid


def fields(p, seed):
    N = p["n"][0] * p["n"][1]
    g = torch.Generator(device="cuda").manual_seed(seed)
    rho = 1 + 1e-2 * torch.randn(N, generator=g, device="cuda", dtype=torch.float64)
    return rho, 2e-2 * torch.randn((2, N), generator=g, device="cuda", dtype=torch.float64)


# one tile, tiles over the whole of x, tiles with a ring on all sides, the ring
# as wide as the domain, a last tile of fewer rows and columns, each tile size
SIZES = [(8, 8), (9, 200), (64, 32), (257, 129), (700, 90), (1031, 517), (2048, 1024)]


@pytest.mark.parametrize("kind", ["periodic", "walls", "solid", "ncde"])
@pytest.mark.parametrize("storage", ["f32dev", "f64"])
@pytest.mark.parametrize("n", SIZES)
def test_passes_equal_single_steps(R, kind, storage, n):
    print(f"[tile steps] {kind} {storage} {n}", file=sys.stderr, flush=True)
    pattern = "AB" if (n[0] + (kind == "solid")) % 2 else "AA"
    p, solid = params(kind, n, storage, pattern)
    ref, dom = (R.Domain(R.make_params(**p), *fields(p, 3), solid=solid) for _ in range(2))
    ref.set_launch(*ref.get_launch())
    for steps in (4, 1, 5, 6, 19, 264):
        ref.step(steps)
        dom.step(steps)
        torch.cuda.synchronize()
        assert torch.equal(ref.populations(), dom.populations()), (steps, dom.steps_taken())
    ref.close()
    dom.close()


@pytest.mark.parametrize("kind,storage,pattern", [("solid", "f32dev", "AA"), ("walls", "f32dev", "AB"), ("periodic", "f64", "AA")])
def test_batches_equal_single_steps(R, kind, storage, pattern):
    print(f"[tile steps batch] {kind} {storage} {pattern}", file=sys.stderr, flush=True)
    made = [params(kind, n, storage, pattern) for n in [(40, 24), (300, 200), (129, 65), (512, 256)]]
    ref, bat = (R.Batch([R.make_params(**p) for p, _ in made], solids=[s for _, s in made]) for _ in range(2))
    ref.set_config(0)
    for b in (ref, bat):
        for k, (p, _) in enumerate(made):
            b.domains[k].set_fields(*fields(p, k))
    for steps in (4, 1, 7, 50):
        ref.step(steps)
        bat.step(steps)
        torch.cuda.synchronize()
        for x, y in zip(ref.domains, bat.domains):
            assert torch.equal(x.populations(), y.populations()), steps
    assert ref.residuals() == bat.residuals()
    ref.close()
    bat.close()


def test_a_large_domain_takes_the_second_buffer(R):
    p, _ = params("periodic", (2048, 2048), "f32dev", "AA")
    dom = R.Domain(R.make_params(**p), *fields(p, 1))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    dom.step(8)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] >= R.population_bytes(dom.params)
    dom.close()
