"""Short calls on rD2Q9 take no passes that are slower than their single steps: a
call of four to ten steps against the same call of a domain that is kept on single
steps (rmrt_set_launch), both timed in turn."""
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


def make(R, n, storage, kind, single):
    p = dict(lattice="Q9", n=(*n, 1), storage=storage, pattern="AA", dx=(1.0, 0.5, 1.0), nu=0.05, rho0=1.0)
    if kind != "periodic":
        p.update(wall_faces=R.WALL_YM | R.WALL_YP)
    if kind == "forced":
        p.update(force=(1e-6, 0.0, 0.0))
    N = n[0] * n[1]
    rho = torch.ones(N, device="cuda", dtype=torch.float64)
    dom = R.Domain(R.make_params(**p), rho, torch.full((2, N), 1e-2, device="cuda", dtype=torch.float64))
    if single:
        dom.set_launch(*dom.get_launch())
    return dom


def seconds(dom, steps, calls):
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(calls):
        dom.step(steps)
    torch.cuda.synchronize()
    return time.perf_counter() - t0


# sizes at which passes of two steps take 1.1 to 1.4 times their single steps
@pytest.mark.parametrize("storage,kind", [("f32dev", "periodic"), ("f32dev", "walls"), ("f32dev", "forced"), ("f64", "walls")])
@pytest.mark.parametrize("n", [(700, 700), (1500, 700), (1500, 1024)])
def test_short_calls_are_no_slower_than_single_steps(R, n, storage, kind):
    for steps in (4, 5, 10):
        dom, ref = make(R, n, storage, kind, False), make(R, n, storage, kind, True)
        best = {id(dom): 1e30, id(ref): 1e30}
        for d in (dom, ref):
            seconds(d, steps, 3)
        for _ in range(6):
            for d in (dom, ref):
                best[id(d)] = min(best[id(d)], seconds(d, steps, 40))
        ratio = best[id(dom)] / best[id(ref)]
        assert ratio < 1.08, (n, storage, kind, steps, ratio)
        dom.close()
        ref.close()
