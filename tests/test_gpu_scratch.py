"""Calls that take their scratch from the buffer that all threads and streams share: captured into a graph (where they
need none) and on two streams at once they give the values of the plain call."""
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


def _eloc(nqs, L, F, n, seed):
    model = nqs.Model.rescnn(L, F, 1, workloads.rescnn_params(F, 1, seed))
    model.prepare("f32")
    ham = nqs.Hamiltonian("tfim", 2, L, 1.0, -1.3, True)
    x = torch.from_numpy(workloads.random_spins(n, L * L, seed)).to(DEV)
    out = torch.zeros(n, dtype=torch.float64, device=DEV)
    return lambda: nqs.nqs_local_energy(model, ham, x, out), [out]


def _grad(nqs, N, widths, n, seed):
    model = nqs.Model("ffnn", N, widths, workloads.ffnn_params(N, widths, seed, 0.1))
    model.prepare("f32")
    x = torch.from_numpy(workloads.random_spins(n, N, seed)).to(DEV)
    lp = torch.zeros(n, dtype=torch.float32, device=DEV)
    O = torch.zeros(n, model.n_params, dtype=torch.float32, device=DEV)
    return lambda: nqs.nqs_logpsi_grad(model, x, logpsi=lp, O=O), [lp, O]


CALLS = {
    "eloc": lambda nqs, s: _eloc(nqs, 4, 16, 40, s),
    "eloc_wide": lambda nqs, s: _eloc(nqs, 5, 32, 30, s),
    "eloc_large": lambda nqs, s: _eloc(nqs, 16, 16, 3, s),                # 256 sites
    "grad": lambda nqs, s: _grad(nqs, 36, (144, 72), 130, s),             # rows of O multiples of 16 bytes
    "grad_odd": lambda nqs, s: _grad(nqs, 25, (131, 67), 63, s),          # odd widths, a tile less one sample
    "grad_three": lambda nqs, s: _grad(nqs, 30, (100, 90, 33), 65, s),    # three layers, a tile and one sample
    "grad_one": lambda nqs, s: _grad(nqs, 64, (260,), 64, s),             # one layer
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_captured_call_gives_the_same_values(nqs, name):
    """Under capture the calls take the one-block-per-sample kernels: also the reference for the batched ones."""
    call, outs = CALLS[name](nqs, 3)
    call()
    torch.cuda.synchronize()
    plain = [o.clone() for o in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for o, p in zip(outs, plain):
            # FP32 values are equal; an energy J diag + h off may take its last rounding in another place
            assert torch.equal(o, p) if o.dtype == torch.float32 else torch.allclose(o, p, rtol=2.0 ** -50, atol=0.0)
        CALLS["grad_three"](nqs, 5)[0]()   # eager work in between


def test_calls_on_two_streams_take_turns(nqs):
    sides = [[CALLS[name](nqs, s) for name in ("grad", "eloc", "grad_odd")] for s in (3, 4)]
    plain = []
    for side in sides:
        for call, _ in side:
            call()
        torch.cuda.synchronize()
        plain.append([[o.clone() for o in outs] for _, outs in side])
    for side in sides:
        for _, outs in side:
            for o in outs:
                o.zero_()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(4):
        for k in range(3):
            for stream, side in zip(streams, sides):
                with torch.cuda.stream(stream):
                    side[k][0]()
    torch.cuda.synchronize()
    for side, want in zip(sides, plain):
        for (_, outs), ws in zip(side, want):
            for o, w in zip(outs, ws):
                assert torch.equal(o, w)
