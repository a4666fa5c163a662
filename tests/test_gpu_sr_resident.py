"""The one-launch conjugate-gradient solve at the edges of its register layouts: the residual in FP64, the same bits
from a second call, and y in the energies' own buffer (which takes the separate launches)."""
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


def _system(n):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    O = torch.randn(n, max(4, n // 3), generator=gen, device=DEV, dtype=torch.float64) + 0.3
    O -= O.mean(dim=0)
    T = (O @ O.T / n).float().contiguous()
    return T, 3.0 * torch.randn(n, generator=gen, device=DEV, dtype=torch.float64) - 100.0


@pytest.mark.parametrize("n", [2, 15, 17, 255, 512, 513, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 5120, 5121])
def test_solve_meets_its_tolerance(nqs, n):
    T, eps = _system(n)
    y = torch.full((n,), float("nan"), dtype=torch.float64, device=DEV)
    its, rel = nqs.nqs_sr_solve(T, eps, 1e-2, y, tol=1e-10, max_iter=2000)
    b = eps - eps.mean()
    r = T.double() @ y + 1e-2 * y - b
    # the recurrence residual that stops the iteration, plus FP64 rounding of the true one
    assert 0 < its and its % 8 == 0 and rel <= 1e-10
    assert float(r.norm() / b.norm()) <= 1e-10 + 1e-11
    again = torch.empty_like(y)
    assert nqs.nqs_sr_solve(T, eps, 1e-2, again, tol=1e-10, max_iter=2000) == (its, rel)
    assert torch.equal(y, again)
    nqs.nqs_sr_solve(T, eps, 1e-2, eps, tol=1e-10, max_iter=2000)
    # two solutions within the tolerance of a system with condition number at most (|T| + 1e-2) / 1e-2
    cond = float(torch.linalg.matrix_norm(T.double(), 1)) / 1e-2 + 1.0
    assert float((eps - y).norm() / y.norm()) <= 3e-10 * cond


def test_iteration_cap_and_constant_energies(nqs):
    T, eps = _system(100)
    y = torch.empty(100, dtype=torch.float64, device=DEV)
    its, rel = nqs.nqs_sr_solve(T, eps, 1e-6, y, tol=1e-14, max_iter=5)
    assert its == 5 and rel > 1e-14
    its, rel = nqs.nqs_sr_solve(T, torch.full_like(eps, 2.0), 1e-6, y)
    assert its == 0 and rel == 0.0 and not torch.any(y)
