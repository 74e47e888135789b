"""Two steps per pass (k_two_step) against single steps of the same library.

The two paths run the same collision with the same roundings, so their
populations agree bit for bit; the single steps are compared with the oracle
elsewhere.  rmrt_set_launch, here with the values a context starts with, keeps
a context on single steps."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2206_00366_amd import rmrt
    return rmrt


def make(R, prm, seed, single=False):
    nx, ny, nz = prm["n"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    rho = 1 + 1e-2 * torch.randn(nx * ny * nz, generator=g, device="cuda", dtype=torch.float64)
    u = 2e-2 * torch.randn((3, nx * ny * nz), generator=g, device="cuda", dtype=torch.float64)
    dom = R.Domain(R.make_params(**prm, nu=0.05, rho0=1.0), rho, u)
    if single:
        dom.set_launch(*dom.get_launch())
    return dom


# whole rows (a last patch of fewer rows, a last chunk of fewer planes), rows
# split along x (with and without whole cache lines), the largest whole row,
# both patterns
CASES = [
    ("Q19", "f32dev", "AA", (128, 128, 96)),
    ("Q19", "f32dev", "AB", (250, 203, 61)),
    ("Q19", "f32dev", "AA", (512, 83, 101)),
    ("Q19", "f32dev", "AA", (1031, 70, 67)),
    ("Q19", "f64", "AB", (128, 128, 96)),
    ("Q19", "f64", "AA", (341, 90, 80)),
    ("Q19", "f64", "AB", (203, 131, 77)),
    ("Q27", "f32dev", "AA", (160, 120, 111)),
    ("Q27", "f32dev", "AB", (341, 121, 96)),
]


@pytest.mark.parametrize("lattice,storage,pattern,n", CASES)
def test_two_steps_per_pass_equal_single_steps(R, lattice, storage, pattern, n):
    print(f"[two-step] {lattice} {storage} {pattern} {n}", file=sys.stderr, flush=True)
    prm = dict(lattice=lattice, storage=storage, pattern=pattern, n=n, dx=(1.0, 1.0, 2.0))
    ref, dom = make(R, prm, 5, single=True), make(R, prm, 5)
    # an even and an odd start, a remainder of each length, a chunk of the graph cache
    for steps in (4, 1, 5, 10, 264):
        ref.step(steps)
        dom.step(steps)
        torch.cuda.synchronize()
        assert torch.equal(ref.populations(), dom.populations()), (steps, dom.steps_taken())
    ref.close()
    dom.close()


def test_the_second_buffer_is_the_contexts_own_and_is_given_back(R):
    prm = dict(lattice="Q19", storage="f32dev", pattern="AA", n=(256, 256, 128), dx=(1.0, 1.0, 2.0))
    dom = make(R, prm, 1)
    size = R.population_bytes(dom.params)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    dom.step(3)     # fewer than four steps: single steps, no second buffer
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < size // 2
    dom.step(4)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] >= size
    dom.close()
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < size // 2


def test_prepared_and_interleaved_streams(R):
    """Two contexts on two streams at once, their graphs prepared beforehand, and a
    source field attached and detached in between (single steps while attached)."""
    prm = dict(lattice="Q19", storage="f32dev", pattern="AA", n=(160, 144, 90), dx=(1.0, 1.0, 2.0))
    refs = [make(R, prm, k, single=True) for k in (2, 3)]
    doms = [make(R, prm, k) for k in (2, 3)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for d, s in zip(doms, streams):
        with torch.cuda.stream(s):
            d.prepare(8)
            d.step(8)
    for r in refs:
        r.step(8)
    torch.cuda.synchronize()
    for r, d in zip(refs, doms):
        assert torch.equal(r.populations(), d.populations())
    F = torch.full((3, doms[0].N), 1e-5, device="cuda")
    for d in (refs[0], doms[0]):
        d.set_source_fields(F=F)
        d.step(8)
        d.set_source_fields()
        d.step(8)
    torch.cuda.synchronize()
    assert torch.equal(refs[0].populations(), doms[0].populations())
    for d in refs + doms:
        d.close()
