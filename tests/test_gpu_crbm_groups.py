"""Complex RBM: the sampler takes whole waves of chains once there are more than one per SIMD, and the local energies run
in groups of samples.  A call equals calls over parts, bit for bit; the largest networks, whose workgroups hold one
sample, are compared with the product of FP64 ratios."""
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


@pytest.mark.parametrize("L,M,sw,trace", [(4, 17, 37, True), (6, 200, 33, False), (7, 300, 5, False), (10, 500, 1, True)])
def test_parts_equal_the_whole(nqs, L, M, sw, trace):
    N, C, S, B = L * L, 2049, 3, 1
    model = nqs.Model("crbm", N, (M,), workloads.crbm_params(N, M, 0.05, 0.05, 3))

    def run(n, offset):
        cfg = nqs.SampleConfig(n_chains=n, n_sweeps=S, n_burnin=B, seed=5, dtype="f16", move="flip", sweep_size=sw,
                               chain_id_offset=offset)
        out = [torch.empty(n, N, dtype=torch.int8, device=DEV), torch.empty(S, n, N, dtype=torch.int8, device=DEV),
               torch.empty(S, n, dtype=torch.float32, device=DEV), torch.empty(n, dtype=torch.int64, device=DEV)]
        nqs.nqs_sample(model, cfg, *out)
        return out

    ham = nqs.Hamiltonian("tfim", 2, L, 1.0, 3.04, True)

    def energies(x):
        er, ei = (torch.empty(x.shape[0], dtype=torch.float64, device=DEV) for _ in range(2))
        nqs.nqs_local_energy_complex(model, ham, x.contiguous(), er, ei, "f16")
        return er, ei

    st, sm, lp, acc = run(C, 0)
    er, ei = energies(sm[S - 1])
    assert torch.all(torch.isfinite(er)) and torch.all(torch.isfinite(ei))
    for at, n in ((0, 1), (1025, 1024), (3, 64), (2048, 1)):
        p_st, p_sm, p_lp, p_acc = run(n, at)
        assert torch.equal(p_st, st[at:at + n]) and torch.equal(p_sm, sm[:, at:at + n])
        assert torch.equal(p_lp, lp[:, at:at + n]) and torch.equal(p_acc, acc[at:at + n])
        p_er, p_ei = energies(sm[S - 1, at:at + n])
        assert torch.equal(p_er, er[at:at + n]) and torch.equal(p_ei, ei[at:at + n])
    model.close()


def test_one_sample_per_workgroup(nqs):
    """20 x 20 sites, 4,200 units: more than 160 KB of LDS for four samples."""
    L, M, n = 20, 4200, 3
    N = L * L
    p = workloads.crbm_params(N, M, 0.004, 0.004, 3)
    model = nqs.Model("crbm", N, (M,), p)
    x = workloads.random_spins(n, N, 2)
    er, ei = (torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(2))
    nqs.nqs_local_energy_complex(model, nqs.Hamiltonian("tfim", 2, L, 1.0, 0.8, True), torch.from_numpy(x).to(DEV), er, ei,
                                 "f32")
    P = N + M + N * M
    z = (p[:P] + 1j * p[P:])
    z = z.real.astype(np.float32).astype(np.float64) + 1j * z.imag.astype(np.float32).astype(np.float64)
    a, b, W = z[:N], z[N:N + M], z[N + M:].reshape(M, N)
    for k in range(n):
        s = x[k].astype(np.float64)
        th = W @ s + b
        lr = -2.0 * a * s + np.array([np.sum(np.log(np.cosh(th - 2.0 * s[i] * W[:, i]) / np.cosh(th))) for i in range(N)])
        g = s.reshape(L, L)
        ref = np.sum(g * np.roll(g, -1, 0)) + np.sum(g * np.roll(g, -1, 1)) + 0.8 * np.sum(np.exp(lr))
        # every factor of a ratio carries at most eight roundings of 2^-24, theta's sum N more that tanh passes on and
        # the column weights by |sinh 2W| (below 0.05)
        bound = 0.8 * np.sum(np.abs(np.exp(lr))) * M * (8 + 0.05 * N) * 2.0 ** -24
        assert abs(er[k].item() + 1j * ei[k].item() - ref) <= bound
    model.close()
