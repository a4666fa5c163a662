"""Log-derivatives of deep wide dense networks, whose factors of one sample together exceed the LDS (eight layers of 2,731
and 2,752 units: 164 and 165 KB), against the outer products of exactly known factors.

Every weight matrix holds one +-1 per row (and per column from the second layer on), so that pre-activations are multiples of
1/4 below 2^10 and exact in FP32, and so is every delta: the last layer's, which its bias block of O holds, moved and
signed.  One multiply per value of O is left, so the values are equal."""
import numpy as np
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


def _network(N, W, L, rng):
    """Parameters, and per layer the column, sign and bias of each row."""
    parts, rows = [], []
    for l in range(L):
        cols = rng.permutation(W) if l else rng.integers(0, N, W)
        sign = rng.choice([-1.0, 1.0], W)
        bias = rng.integers(-4, 8, W) / 4.0
        w = np.zeros((W, W if l else N))
        w[np.arange(W), cols] = sign
        parts += [w.reshape(-1), bias]
        rows.append((cols, sign.astype(np.float32), bias.astype(np.float32)))
    return np.concatenate(parts), rows


@pytest.mark.parametrize("W", [2752, 2731])
def test_factors_beyond_the_lds(nqs, W):
    N, L, n = 64, 8, 3
    rng = np.random.default_rng(W)
    p, rows = _network(N, W, L, rng)
    model = nqs.Model("ffnn", N, (W,) * L, p)
    P = model.n_params
    del p
    x = (2 * rng.integers(0, 2, (n, N)) - 1).astype(np.int8)
    xd = torch.from_numpy(x).to(DEV)
    O = torch.full((n, P), float("nan"), dtype=torch.float32, device=DEV)
    nqs.nqs_logpsi_grad(model, xd, O=O)

    acts = [x.astype(np.float32)]
    for cols, sign, bias in rows:
        acts.append(np.maximum(acts[-1][:, cols] * sign + bias, np.float32(0)))
    delta = O[:, P - W:].cpu().numpy()
    assert np.all(np.abs(delta) <= 1.0) and np.count_nonzero(delta) > n * W // 2
    last = acts[-2][:, rows[-1][0]] * rows[-1][1] + rows[-1][2]
    assert np.allclose(delta, np.tanh(last.astype(np.float64)), rtol=0, atol=2.0 ** -21)
    off = [0]
    for l in range(L):
        off.append(off[-1] + W * (W if l else N) + W)
    assert off[-1] == P
    for l in range(L - 1, -1, -1):
        nin = W if l else N
        d, a = torch.from_numpy(delta).to(DEV), torch.from_numpy(acts[l]).to(DEV)
        assert torch.equal(O[:, off[l]:off[l] + W * nin].view(n, W, nin), d[:, :, None] * a[:, None, :])
        assert torch.equal(O[:, off[l] + W * nin:off[l + 1]], d)
        cols, sign, _ = rows[l]
        back = np.zeros((n, nin), dtype=np.float32)
        if l:
            back[:, cols] = delta * sign
            delta = np.where(acts[l] > 0, back, np.float32(0))

    # columns: within a layer, over the end of the first layer, of a layer between and of the last, one value
    for p0, p1 in ((8, 4008), (off[1] - 9000, off[1] + 9000), (off[4] - 30001, off[4] + 3), (P - 20000, P),
                   (off[3] - 1, off[3]), (off[2] - W, off[2])):
        cut = torch.full((n, p1 - p0), float("nan"), dtype=torch.float32, device=DEV)
        nqs.nqs_logpsi_grad_cols(model, xd, p0, p1, cut)
        assert torch.equal(cut, O[:, p0:p1])
    # T over one block of columns is the Gram matrix of O itself
    T, G = (torch.empty(n, n, dtype=torch.float32, device=DEV) for _ in range(2))
    nqs.nqs_gram(O, 1, G)
    nqs.nqs_sample_gram(model, xd, T, P)
    assert torch.equal(T, G)
    model.close()


@pytest.mark.parametrize("N,widths,n", [(25, (100, 50), 2048), (25, (100, 50), 2049), (36, (144, 72), 513), (5, (3,), 70),
                                            (64, (256, 128), 300), (40, (64, 404, 32), 70)])
def test_columns_equal_the_whole(nqs, N, widths, n):
    """Few samples and columns take one block per sample, others the factors: the values do not depend on it."""
    rng = np.random.default_rng(n)
    sizes = [N, *widths]
    P = sum(o * (i + 1) for i, o in zip(sizes, sizes[1:]))
    model = nqs.Model("ffnn", N, widths, rng.normal(scale=0.1, size=P))
    x = torch.from_numpy((2 * rng.integers(0, 2, (n, N)) - 1).astype(np.int8)).to(DEV)
    O = torch.empty(n, P, dtype=torch.float32, device=DEV)
    nqs.nqs_logpsi_grad(model, x, O=O)
    for p0, p1 in ((0, P), (0, P - 1), (P // 3, P // 3 + 1), (1, P // 16 + 1), (2, 2 + P // 4), (P // 2, P)):
        cut = torch.full((n, p1 - p0), float("nan"), dtype=torch.float32, device=DEV)
        nqs.nqs_logpsi_grad_cols(model, x, p0, p1, cut)
        assert torch.equal(cut, O[:, p0:p1])
    model.close()
