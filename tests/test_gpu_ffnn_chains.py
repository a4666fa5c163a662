"""The two-layer dense sampler takes eight, four, two or one chains per wave by the number of chains.  A call over many
chains equals calls over fewer, which run with fewer chains per wave, bit for bit: last waves and blocks that are only
partly filled, the fewest and most first-layer units of the register-resident kernel, both moves, traces."""
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


@pytest.mark.parametrize("N,widths,move,dtype", [
    (36, (144, 72), "exchange", "bf16"), (36, (144, 72), "flip", "bf16"), (16, (512, 200), "exchange", "f16"),
    (34, (67, 33), "exchange", "f16"), (9, (75, 64), "flip", "f16")])
def test_many_chains_equal_fewer(nqs, N, widths, move, dtype):
    model = nqs.Model("ffnn", N, widths, workloads.ffnn_params(N, widths, 3, 0.05))
    C, S, B = 16401, 4, 1

    def run(n, offset):
        cfg = nqs.SampleConfig(n_chains=n, n_sweeps=S, n_burnin=B, seed=5, dtype=dtype, move=move, refresh_sweeps=2,
                               sweep_size=12, chain_id_offset=offset)
        out = [torch.empty(n, N, dtype=torch.int8, device=DEV), torch.empty(S, n, N, dtype=torch.int8, device=DEV),
               torch.empty(S, n, dtype=torch.float32, device=DEV), torch.empty(n, dtype=torch.int64, device=DEV)]
        nqs.nqs_sample(model, cfg, *out)
        return out

    st, sm, lp, acc = run(C, 0)
    for at, n in ((8205, 8196), (3, 4097), (16400, 1), (16384, 17), (1001, 2047), (5, 2049)):
        p_st, p_sm, p_lp, p_acc = run(n, at)
        assert torch.equal(p_st, st[at:at + n])
        assert torch.equal(p_sm, sm[:, at:at + n])
        assert torch.equal(p_lp, lp[:, at:at + n])
        assert torch.equal(p_acc, acc[at:at + n])
    model.close()
