"""RBM sampler: proposals are read ahead of the decision they follow, across the ends of batches and sweeps.  One call
equals its sweeps run one call at a time (each starts the read-ahead anew), bit for bit: few sites, so that a site is
often proposed twice running, sweeps of one step, of whole batches and of neither, every number of lanes per chain."""
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


@pytest.mark.parametrize("N,M,G", [(2, 3, 16), (3, 40, 32), (5, 70, 64), (33, 200, 16), (40, 1000, 64)])
@pytest.mark.parametrize("sw", [1, 7, 16, 65])
def test_one_call_equals_its_sweeps(nqs, N, M, G, sw):
    model = nqs.Model("rbm", N, (M,), workloads.rbm_params(N, M, 0.1, 3))
    C, S = 130, 5

    def run(n_sweeps, offset, state):
        cfg = nqs.SampleConfig(n_chains=C, n_sweeps=n_sweeps, n_burnin=0, seed=5, dtype="f32", move="flip", sweep_size=sw,
                               lanes_per_chain=G, refresh_sweeps=1, step_offset=offset, init_chains=state is None)
        st = torch.empty(C, N, dtype=torch.int8, device=DEV) if state is None else state.clone()
        sm = torch.empty(n_sweeps, C, N, dtype=torch.int8, device=DEV)
        acc = torch.empty(C, dtype=torch.int64, device=DEV)
        nqs.nqs_sample(model, cfg, st, sm, None, acc)
        return st, sm, acc

    w_st, w_sm, w_acc = run(S, 0, None)
    st, acc = None, torch.zeros(C, dtype=torch.int64, device=DEV)
    for q in range(S):
        st, sm, a = run(1, q * sw, st)
        acc += a
        assert torch.equal(sm[0], w_sm[q])
    assert torch.equal(st, w_st) and torch.equal(acc, w_acc)
    model.close()
