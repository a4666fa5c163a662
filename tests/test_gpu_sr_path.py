"""Which path nqs_sr_solve takes: one launch up to 5,120 unknowns (every register layout), separate launches beyond, for one
unknown, for y in the energies' buffer, and after a block of the one launch gave up waiting, with the same solution."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def nqs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_20782_amd as m
    m.load()
    return m


@pytest.fixture
def lib(nqs):
    lib = nqs.load()
    yield lib
    lib.nqs_probe_solve_polls(0)


def _system(n):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    O = torch.randn(n, max(4, n // 3), generator=gen, device=DEV, dtype=torch.float64) + 0.3
    O -= O.mean(dim=0)
    return (O @ O.T / n).float().contiguous(), 3.0 * torch.randn(n, generator=gen, device=DEV, dtype=torch.float64) - 100.0


def _residual(T, eps, y):
    b = eps - eps.mean()
    return float((T.double() @ y + 1e-2 * y - b).norm() / b.norm())


@pytest.mark.parametrize("n,one", [(1, 0), (2, 1), (512, 1), (513, 1), (1025, 1), (2049, 1), (4096, 1), (4097, 1), (5120, 1),
                                   (5121, 0)])
def test_path_by_size(nqs, lib, n, one):
    T, eps = _system(n)
    y = torch.empty_like(eps)
    nqs.nqs_sr_solve(T, eps, 1e-2, y, tol=1e-10, max_iter=2000)
    assert lib.nqs_probe_solve_one_launch() == one
    nqs.nqs_sr_solve(T, eps, 1e-2, eps, tol=1e-10, max_iter=2000)
    assert lib.nqs_probe_solve_one_launch() == 0


@pytest.mark.parametrize("n", [600, 4096, 5000])
def test_fallback_after_a_wait_that_gives_up(nqs, lib, n):
    T, eps = _system(n)
    y, z = torch.empty_like(eps), torch.empty_like(eps)
    lib.nqs_probe_solve_polls(1)   # the first blocks there find the others' slots empty
    its, rel = nqs.nqs_sr_solve(T, eps, 1e-2, y, tol=1e-10, max_iter=2000)
    assert lib.nqs_probe_solve_one_launch() == 0
    # the recurrence residual that stops the iteration, plus FP64 rounding of the true one
    assert 0 < its and rel <= 1e-10 and _residual(T, eps, y) <= 1e-10 + 1e-11
    lib.nqs_probe_solve_polls(0)
    nqs.nqs_sr_solve(T, eps, 1e-2, z, tol=1e-10, max_iter=2000)
    assert lib.nqs_probe_solve_one_launch() == 1 and _residual(T, eps, z) <= 1e-10 + 1e-11
