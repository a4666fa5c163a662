"""The batched dense-network sampler: one call over many chains, whose matrix products run in large tiles, equals calls
over a few chains at a time (small tiles, other rows, other blocks of chains) bit for bit.  The sizes choose each tile
of the products, widths and sites that end inside a block, spins past the last piece, an odd number of sites per sweep
and more chains than one pass over the counts covers."""
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


@pytest.mark.parametrize("N,widths,C,piece,move,dtype", [
    (65, (390, 270, 129), 16001, 999, "flip", "bf16"), (65, (390, 270, 129), 40000, 4001, "flip", "f16"),
    (65, (390, 270, 129), 32001, 4001, "flip", "e4m3"), (100, (420, 430), 24000, 2000, "exchange", "bf16"),
    (100, (420, 430), 24000, 2000, "flip", "bf16"), (33, (70, 430), 16001, 2000, "flip", "e4m3"),
    (7, (9, 5, 3), 270001, 64, "flip", "bf16"), (12, (9, 65), 130, 1, "exchange", "e4m3"),
    (20, (31, 64, 9), 300, 65, "exchange", "f32")])
def test_many_chains_equal_few_at_a_time(nqs, N, widths, C, piece, move, dtype):
    model = nqs.Model("ffnn", N, widths, workloads.ffnn_params(N, widths, 3, 0.05))
    S, B, sw = 2, 1, 3

    def run(n, offset, **kw):
        cfg = nqs.SampleConfig(n_chains=n, n_sweeps=S, n_burnin=B, sweep_size=sw, seed=5, dtype=dtype, move=move,
                               lanes_per_chain=-1, chain_id_offset=offset, **kw)
        out = [torch.empty(n, N, dtype=torch.int8, device=DEV), torch.empty(S, n, N, dtype=torch.int8, device=DEV),
               torch.empty(S, n, dtype=torch.float32, device=DEV), torch.empty(n, dtype=torch.int64, device=DEV)]
        nqs.nqs_sample(model, cfg, *out)
        return out

    st, sm, lp, acc = run(C, 0)
    starts = [0, (C // 2 // piece) * piece, C - min(piece, C % piece or piece)]
    for at in starts:
        n = min(piece, C - at)
        p_st, p_sm, p_lp, p_acc = run(n, at)
        assert torch.equal(p_st, st[at:at + n])
        assert torch.equal(p_sm, sm[:, at:at + n])
        assert torch.equal(p_lp, lp[:, at:at + n])
        assert torch.equal(p_acc, acc[at:at + n])
    assert torch.all(acc >= 0) and torch.all(acc <= (S + B) * sw)
    model.close()
