"""The first call of four steps or more sets its passes up in stream order: it does
not wait for the work queued before it."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2206_00366_amd import rmrt
    return rmrt


FORMS = [("Q9", "f32dev", (2048, 2048, 1)), ("Q19", "f32dev", (128, 128, 128))]


def domain(R, lattice, storage, n, pattern="AA"):
    N = n[0] * n[1] * n[2]
    p = R.make_params(lattice=lattice, storage=storage, pattern=pattern, n=n, nu=0.05, rho0=1.0)
    return R.Domain(p, torch.ones(N, device="cuda", dtype=torch.float64),
                    torch.full((2 if n[2] == 1 else 3, N), 1e-2, device="cuda", dtype=torch.float64))


def batch(R, lattice, storage, n, pattern="AA"):
    return R.Batch([R.make_params(lattice=lattice, storage=storage, pattern=pattern, n=n, nu=0.05, rho0=1.0)] * 2)


def still_running_after(fn):
    """Did the call return before the second or so of work queued ahead of it was done?"""
    a = torch.ones(8192, 8192, device="cuda")
    out = torch.empty_like(a)
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    each = time.perf_counter() - t0
    for _ in range(int(1.0 / each) + 1):
        torch.mm(a, a, out=out)
    ev = torch.cuda.Event()
    ev.record()
    fn()
    running = not ev.query()
    torch.cuda.synchronize()
    return running


@pytest.mark.parametrize("pattern", ["AA", "AB"])
@pytest.mark.parametrize("kind", ["tiles", "sweep", "batch"])
def test_the_first_call_does_not_wait_for_the_stream(R, kind, pattern):
    make = batch if kind == "batch" else domain
    warm, ref, dom = (make(R, *FORMS[kind == "sweep"], pattern=pattern) for _ in range(3))
    warm.step(8)    # loads the kernels
    ref.step(8)
    assert still_running_after(lambda: dom.step(8))
    pairs = zip(ref.domains, dom.domains) if kind == "batch" else [(ref, dom)]
    for x, y in pairs:
        assert torch.equal(x.populations(), y.populations())
    for d in (warm, ref, dom):
        d.close()
