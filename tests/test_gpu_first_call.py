"""The second buffer of the first call of four steps or more: not for domains and
batches that take single steps only."""
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


def taken(fn):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    fn()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("lattice,storage,n", FORMS)
def test_a_domain_on_single_steps_takes_no_second_buffer(R, lattice, storage, n):
    dom = domain(R, lattice, storage, n)
    size = R.population_bytes(dom.params)
    dom.set_launch(*dom.get_launch())
    assert taken(lambda: dom.step(8)) < size // 2
    dom.tune(4)     # back on passes, which are set up now
    assert taken(lambda: dom.step(8)) >= size
    dom.close()


@pytest.mark.parametrize("pin", ["set_config", "set_group_bytes", "set_xcd_chunks"])
def test_a_batch_on_single_steps_takes_no_second_buffer(R, pin):
    b = batch(R, *FORMS[0])
    size = 2 * R.population_bytes(b.params[0])
    getattr(b, pin)(0)
    assert taken(lambda: b.step(8)) < size // 2
    b.close()
