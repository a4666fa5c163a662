"""Dense and RBM calls over more samples than one piece of their factors holds: the number of 64-sample tiles that a grid
takes (65,535, for the narrowest networks) and the scratch memory cut the samples into chunks.  log|psi| and O equal the
same calls over parts bit for bit, the vector-Jacobian product is the FP64 sum over O."""
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


@pytest.mark.parametrize("arch,N,widths,n", [
    ("ffnn", 8, (4,), 65536 * 64 + 65),          # one tile and one sample more than a grid holds, 12 values a sample
    ("ffnn", 8, (4,), 65535 * 64 + 1),
    ("ffnn", 4, (3999,), 16865), ("ffnn", 3, (3000, 2), 11300), ("rbm", 4, (1000,), 67141)])
def test_chunks_of_samples(nqs, arch, N, widths, n):
    p = workloads.rbm_params(N, widths[0], 0.1, 3) if arch == "rbm" else workloads.ffnn_params(N, widths, 3, 0.1)
    model = nqs.Model(arch, N, widths, p)
    P = model.n_params
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    x = (2 * torch.randint(0, 2, (n, N), generator=gen, device=DEV, dtype=torch.int8) - 1).contiguous()
    g = torch.randn(n, generator=gen, device=DEV)
    lp = torch.full((n,), float("nan"), dtype=torch.float32, device=DEV)
    O = torch.full((n, P), float("nan"), dtype=torch.float32, device=DEV)
    vjp = torch.full((P,), float("nan"), dtype=torch.float32, device=DEV)
    nqs.nqs_logpsi_grad(model, x, logpsi=lp, O=O, vjp_in=g, vjp_out=vjp)
    step = 4000 if P > 1000 else 1000003
    ref = torch.zeros(P, dtype=torch.float64, device=DEV)
    size = torch.zeros(P, dtype=torch.float64, device=DEV)
    for at in range(0, n, step):
        m = min(step, n - at)
        plp = torch.empty(m, dtype=torch.float32, device=DEV)
        pO = torch.empty(m, P, dtype=torch.float32, device=DEV)
        nqs.nqs_logpsi_grad(model, x[at:at + m], logpsi=plp, O=pO)
        assert torch.equal(plp, lp[at:at + m]) and torch.equal(pO, O[at:at + m])
        terms = g[at:at + m].double().unsqueeze(1) * pO.double()
        ref += terms.sum(dim=0)
        size += terms.abs().sum(dim=0)
    # O's values are rounded to FP32 (2^-24 each), the result once more, and n FP64 additions on either side
    bound = (2.0 ** -23 + 2 * n * 2.0 ** -53) * size + 1e-30
    assert torch.all((vjp.double() - ref).abs() <= bound)
    model.close()
