"""Local energies of the two-layer dense network in 16 bits: the samples of a call are evaluated in groups whose size
follows their number and the LDS.  A call equals calls over parts of its samples, in other groups, bit for bit: TFIM and
Heisenberg rows, one and two dimensions, open boundaries, the fewest and most first-layer units."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def nqs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_20782_amd as m
    m.load()
    return m


@pytest.mark.parametrize("kind,dim,L,pbc,widths,dtype", [
    ("heisenberg", 2, 6, True, (144, 72), "bf16"), ("tfim", 2, 6, False, (131, 200), "f16"),
    ("heisenberg", 1, 18, True, (67, 33), "f16"), ("tfim", 1, 9, True, (512, 130), "bf16"),
    ("heisenberg", 2, 10, True, (400, 200), "f16")])
def test_parts_of_the_samples(nqs, kind, dim, L, pbc, widths, dtype):
    N, n = L ** dim, 3100
    model = nqs.Model("ffnn", N, widths, workloads.ffnn_params(N, widths, 3, 0.05))
    ham = nqs.Hamiltonian(kind, dim, L, 1.0, 0.7, pbc)
    x = torch.from_numpy(workloads.random_spins(n, N, 2)).to(DEV)
    whole = torch.empty(n, dtype=torch.float64, device=DEV)
    nqs.nqs_local_energy(model, ham, x, whole, dtype)
    assert torch.all(torch.isfinite(whole))
    for at, m in ((0, 1), (7, 255), (1000, 257), (500, 600), (900, 2111)):
        part = torch.empty(m, dtype=torch.float64, device=DEV)
        nqs.nqs_local_energy(model, ham, x[at:at + m].contiguous(), part, dtype)
        assert torch.equal(part, whole[at:at + m])
    model.close()
