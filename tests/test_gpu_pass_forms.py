"""Every form of the rD2Q9 passes (storage x equation x constant source x walls and
solid nodes) against single steps of the same library, bit for bit; the forms that
have no pass; and that the comparisons of passes with single steps, here and in
test_gpu_tile_steps.py and test_gpu_two_step.py, are not of single steps with
themselves."""
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


WALLS = {"periodic": 0, "x": 3, "y": 12, "box": 15, "one": 4, "solid": 0, "solid_y": 12}


def make(R, storage, eq, source, bounds, n, pattern, single):
    p = dict(lattice="Q9", storage=storage, pattern=pattern, n=(*n, 1), dx=(1.0, 0.5, 1.0), wall_faces=WALLS[bounds])
    if eq == "NSE":
        p.update(nu=0.05, rho0=1.0, force=(1e-4, 2e-5, 0.0) if source else (0.0, 0.0, 0.0))
    else:
        p.update(equation="NCDE", D0=0.05, D2=0.5, adv=(0.02, 0.01, 0.0), rho0=0.5, source=1e-4 if source else 0.0)
    N = n[0] * n[1]
    g = torch.Generator(device="cuda").manual_seed(n[0])
    rho = 1 + 1e-2 * torch.randn(N, generator=g, device="cuda", dtype=torch.float64)
    u = 2e-2 * torch.randn((2, N), generator=g, device="cuda", dtype=torch.float64)
    solid = (np.random.default_rng(n[1]).random(N) < 0.1).astype(np.uint8) if bounds.startswith("solid") else None
    dom = R.Domain(R.make_params(**p), rho, u if eq == "NSE" else None, solid=solid)
    if single:
        dom.set_launch(*dom.get_launch())
    return dom


@pytest.mark.parametrize("bounds", sorted(WALLS))
@pytest.mark.parametrize("source", [False, True])
@pytest.mark.parametrize("eq", ["NSE", "NCDE"])
@pytest.mark.parametrize("storage", ["f32dev", "f64", "f16dev"])
def test_passes_equal_single_steps(R, storage, eq, source, bounds):
    passes = bounds != "one" and (storage == "f32dev" or (storage == "f64" and not source))
    for n, pattern in (((61, 40), "AA"), ((530, 301), "AB")):
        print(f"[pass forms] {storage} {eq} {source} {bounds} {n}", file=sys.stderr, flush=True)
        ref = make(R, storage, eq, source, bounds, n, pattern, True)
        dom = make(R, storage, eq, source, bounds, n, pattern, False)
        for steps in (8, 1, 6, 4, 23):
            ref.step(steps)
            dom.step(steps)
            torch.cuda.synchronize()
            # (a wall on one of two opposite faces leaves the order of some writes open)
            assert bounds == "one" or torch.equal(ref.populations(), dom.populations()), (n, steps)
            assert ref.step_launches(23) == 23 and (dom.step_launches(23) < 23) == passes
        ref.close()
        dom.close()


@pytest.mark.parametrize("kind", ["periodic", "walls", "solid", "ncde"])
@pytest.mark.parametrize("storage", ["f32dev", "f64"])
def test_the_compared_domains_take_passes(R, storage, kind):
    import test_gpu_tile_steps as T
    for n in T.SIZES:
        p, solid = T.params(kind, n, storage, "AA")
        dom = R.Domain(R.make_params(**p), *T.fields(p, 3), solid=solid)
        assert dom.step_launches(264) == 264
        dom.prepare(264)
        assert dom.step_launches(264) <= 72, n
        dom.close()


def test_the_compared_batches_take_passes(R):
    import test_gpu_tile_steps as T
    for kind, storage, pattern in [("solid", "f32dev", "AA"), ("walls", "f32dev", "AB"), ("periodic", "f64", "AA")]:
        made = [T.params(kind, n, storage, pattern) for n in [(40, 24), (300, 200), (129, 65), (512, 256)]]
        b = R.Batch([R.make_params(**p) for p, _ in made], solids=[s for _, s in made])
        b.prepare(50)
        assert b.step_launches(50) <= 14
        b.close()


def test_the_compared_3d_domains_take_passes(R):
    import test_gpu_two_step as T
    for lattice, storage, pattern, n in T.CASES:
        dom = T.make(R, dict(lattice=lattice, storage=storage, pattern=pattern, n=n, dx=(1.0, 1.0, 2.0)), 5)
        dom.prepare(264)
        assert dom.step_launches(264) == 128 + 4, (lattice, storage, n)
        dom.close()
