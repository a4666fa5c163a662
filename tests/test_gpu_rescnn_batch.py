"""The convolutional network's batched forward pass at the edges of its batches: rows that fill no tile, a last
workgroup with fewer configurations, one configuration per workgroup against several.  How the configurations are
dealt to workgroups must not change a value, so a call is compared bit for bit with the same work in pieces, and the
local energies with the oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle import rescnn

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def nqs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_20782_amd as m
    m.load()
    return m


def _sample(nqs, model, N, C, dtype, first, seed=3):
    cfg = nqs.SampleConfig(n_chains=C, n_sweeps=2, n_burnin=1, seed=seed, dtype=dtype, chain_id_offset=first)
    state = torch.empty(C, N, dtype=torch.int8, device=DEV)
    samples = torch.empty(2, C, N, dtype=torch.int8, device=DEV)
    logpsi = torch.empty(2, C, dtype=torch.float32, device=DEV)
    acc = torch.empty(C, dtype=torch.int64, device=DEV)
    nqs.nqs_sample(model, cfg, state, samples, logpsi, acc)
    return [t.cpu().numpy() for t in (state, samples, logpsi, acc)]


@pytest.mark.parametrize("dtype,L,F,R,C", [("bf16", 4, 16, 2, 1100), ("f16", 5, 32, 1, 1100), ("f32", 5, 16, 1, 1100),
                                           ("bf16", 10, 16, 1, 600), ("f32", 4, 32, 1, 1025), ("bf16", 3, 32, 0, 16)])
def test_sampler_does_not_depend_on_the_batch(nqs, dtype, L, F, R, C):
    N = L * L
    model = nqs.Model.rescnn(L, F, R, workloads.rescnn_params(F, R, 7 + L))
    whole = _sample(nqs, model, N, C, dtype, 0)
    assert 0 < whole[3].sum() < C * 3 * N
    cut = [0, 1, min(300, C // 2), C]
    parts = [_sample(nqs, model, N, b - a, dtype, a) for a, b in zip(cut, cut[1:])]
    for k, axis in enumerate((0, 1, 1, 0)):
        assert np.array_equal(whole[k], np.concatenate([p[k] for p in parts], axis=axis))


@pytest.mark.parametrize("dtype,L,F,R,n", [("f32", 4, 16, 2, 61), ("bf16", 4, 32, 1, 61), ("f32", 10, 32, 1, 11),
                                           ("f16", 5, 16, 1, 50), ("f32", 3, 16, 0, 1)])
def test_local_energy_does_not_depend_on_the_batch(nqs, dtype, L, F, R, n):
    N, J, h = L * L, 1.0, -1.3
    p = workloads.rescnn_params(F, R, 5 + L)
    model = nqs.Model.rescnn(L, F, R, p)
    ham = nqs.Hamiltonian("tfim", 2, L, J, h, True)
    x = torch.from_numpy(workloads.random_spins(n, N, 3)).to(DEV)
    whole = torch.empty(n, dtype=torch.float64, device=DEV)
    nqs.nqs_local_energy(model, ham, x, whole, dtype)
    one = torch.empty_like(whole)
    for k in range(n):
        nqs.nqs_local_energy(model, ham, x[k:k + 1], one[k:k + 1], dtype)
    assert torch.equal(whole, one)
    if dtype == "f32":
        # the tolerance of the one-configuration kernel's test
        ref = rescnn.ResCNN(L, F, R, p, "f32").local_energy_tfim(x.cpu().numpy(), J, h)
        scale = np.abs(J) * 2 * N + np.abs(h) * np.abs(ref) + 1.0
        assert np.all(np.abs(whole.cpu().numpy() - ref) <= 1e-4 * scale)
