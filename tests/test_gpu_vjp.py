"""The vector-Jacobian product from the factors of O, at the edges of its tiles and sample ranges, against the FP64
sum over O itself."""
import numpy as np
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
    ("rbm", 16, (16,), 1), ("rbm", 63, (64,), 33), ("rbm", 64, (63,), 700), ("rbm", 65, (130,), 129),
    ("ffnn", 10, (7,), 31), ("ffnn", 64, (63, 65), 200), ("ffnn", 36, (144, 72), 1000), ("ffnn", 20, (33, 64, 9), 65)])
def test_vjp_matches_the_sum_over_O(nqs, arch, N, widths, n):
    p = workloads.rbm_params(N, widths[0], 0.1, 3) if arch == "rbm" else workloads.ffnn_params(N, widths, 3, 0.1)
    model = nqs.Model(arch, N, widths, p)
    P = model.n_params
    x = torch.from_numpy(workloads.random_spins(n, N, 2)).to(DEV)
    g = torch.from_numpy(np.random.default_rng(4).normal(size=n).astype(np.float32)).to(DEV)
    O = torch.empty(n, P, dtype=torch.float32, device=DEV)
    out = torch.full((P,), float("nan"), dtype=torch.float32, device=DEV)
    nqs.nqs_logpsi_grad(model, x, O=O)
    nqs.nqs_logpsi_grad(model, x, vjp_in=g, vjp_out=out)
    o64, g64 = O.double(), g.double().unsqueeze(1)
    ref = (g64 * o64).sum(dim=0)
    # O's values are rounded to FP32 (2^-24 each), the result once more; the FP64 sums add nothing at this scale
    bound = 2.0 ** -23 * (g64.abs() * o64.abs()).sum(dim=0) + 1e-30
    assert torch.all((out.double() - ref).abs() <= bound)
    again = torch.empty_like(out)
    nqs.nqs_logpsi_grad(model, x, vjp_in=g, vjp_out=again)
    assert torch.equal(out, again)


@pytest.mark.parametrize("n,P", [(1, 4), (7, 8), (9, 1023), (64, 1024), (100, 1028), (1000, 4097), (513, 7)])
def test_forces_at_row_and_slice_edges(nqs, n, P):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n * P)
    O = torch.randn(n, P, generator=gen, device=DEV)
    e = 3.0 * torch.randn(n, generator=gen, dtype=torch.float64, device=DEV) - 50.0
    F = torch.empty(P, dtype=torch.float64, device=DEV)
    mean = torch.empty(P, dtype=torch.float64, device=DEV)
    nqs.nqs_forces(O, e, F, mean)
    o = O.double()
    # FP64 sums of n terms each: n 2^-53 of the sums of absolute values, here and in the reference
    tol = 2.0 * (n + 4) * 2.0 ** -53
    assert torch.all((mean - o.mean(dim=0)).abs() <= tol * o.abs().mean(dim=0) + 1e-300)
    want = (o * e.unsqueeze(1)).mean(dim=0) - o.mean(dim=0) * e.mean()
    assert torch.all((F - want).abs() <= 3.0 * tol * (o.abs() * e.abs().unsqueeze(1)).mean(dim=0) + tol * o.abs().mean(dim=0) * e.abs().mean() * 3.0)
