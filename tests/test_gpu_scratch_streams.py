"""Calls that work in the library's scratch buffers (log-derivatives of dense networks, local energies of convolutional
ones) on several streams: one stream's call does not wait for another's, neither on the device nor on the host, more
streams than buffers still give the values of the plain call, from one thread or several, and a call is accepted while
another stream is being captured."""
import threading

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


def _eloc(nqs, n, seed):
    model = nqs.Model.rescnn(4, 16, 1, workloads.rescnn_params(16, 1, seed))
    model.prepare("f32")
    ham = nqs.Hamiltonian("tfim", 2, 4, 1.0, -1.3, True)
    x = torch.from_numpy(workloads.random_spins(n, 16, seed)).to(DEV)
    out = torch.zeros(n, dtype=torch.float64, device=DEV)
    return model, out, lambda: nqs.nqs_local_energy(model, ham, x, out)


def _logpsi(nqs, n, seed):
    model = nqs.Model("ffnn", 36, (144, 72), workloads.ffnn_params(36, (144, 72), seed, 0.1))
    model.prepare("f32")
    x = torch.from_numpy(workloads.random_spins(n, 36, seed)).to(DEV)
    out = torch.zeros(n, dtype=torch.float32, device=DEV)
    return model, out, lambda: nqs.nqs_logpsi_grad(model, x, logpsi=out)


def _long_run(nqs):
    """A few waves that keep a stream busy for some tenths of a second and leave nearly all of the GPU free."""
    model = nqs.Model("rbm", 64, (64,), workloads.rbm_params(64, 64, 0.05, 1))
    model.prepare("f32")
    state = torch.ones(4, 64, dtype=torch.int8, device=DEV)
    cfg = nqs.SampleConfig(n_chains=4, n_sweeps=0, n_burnin=20000, seed=1, dtype="f32", move="flip")
    return model, lambda: nqs.nqs_sample(model, cfg, state, None)


def _overlaps(a, b, occupy, call_a, call_b):
    """Whether call_b on stream b ends while stream a is still busy with `occupy` and then call_a."""
    torch.cuda.synchronize()
    end_a, end_b = torch.cuda.Event(), torch.cuda.Event()
    with torch.cuda.stream(a):
        occupy()
        call_a()
        end_a.record()
    with torch.cuda.stream(b):
        call_b()
        end_b.record()
    end_b.synchronize()
    busy = not end_a.query()
    torch.cuda.synchronize()
    return busy


@pytest.mark.parametrize("make,n_a,n_b", [(_eloc, 40, 40), (_eloc, 40, 200000), (_logpsi, 5000, 5000),
                                          (_logpsi, 5000, 160000)])
def test_streams_do_not_wait_for_each_other(nqs, make, n_a, n_b):
    busy_model, occupy = _long_run(nqs)
    side_a, side_b = make(nqs, n_a, 3), make(nqs, n_b, 4)
    x = torch.zeros(64, device=DEV)
    occupy()
    side_a[2]()
    torch.cuda.synchronize()
    # two streams whose work the device runs side by side (streams may share a hardware queue)
    a = torch.cuda.Stream()
    for _ in range(8):
        b = torch.cuda.Stream()
        if _overlaps(a, b, occupy, lambda: None, lambda: x.add_(1.0)):
            break
    else:
        pytest.skip("no two streams run side by side")
    assert _overlaps(a, b, occupy, side_a[2], side_b[2])
    for m in (busy_model, side_a[0], side_b[0]):
        m.close()


@pytest.mark.parametrize("threads", [False, True])
def test_more_streams_than_buffers(nqs, threads):
    sides = [make(nqs, n, s) for s, (make, n) in enumerate(2 * [(_eloc, 50), (_logpsi, 4000), (_eloc, 90), (_logpsi, 900),
                                                               (_eloc, 7), (_logpsi, 2500)])]
    want = []
    for _, out, call in sides:
        call()
        torch.cuda.synchronize()
        want.append(out.clone())
        out.zero_()
    streams = [torch.cuda.Stream() for _ in sides]
    torch.cuda.synchronize()
    errors = []

    def run(k):
        try:
            with torch.cuda.stream(streams[k]):
                for _ in range(4):
                    sides[k][2]()
        except Exception as e:   # noqa: BLE001 (reported below)
            errors.append(e)

    if threads:
        pool = [threading.Thread(target=run, args=(k,)) for k in range(len(sides))]
        for t in pool:
            t.start()
        for t in pool:
            t.join()
    else:
        for k in range(len(sides)):
            run(k)
    torch.cuda.synchronize()
    assert not errors
    for (model, out, _), w in zip(sides, want):
        assert torch.equal(out, w)
        model.close()


def test_accepted_while_another_stream_is_captured(nqs):
    model, out, call = _logpsi(nqs, 130000, 3)
    x = torch.zeros(64, device=DEV)
    streams = [torch.cuda.Stream() for _ in range(9)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):           # global capture mode
        x.add_(1.0)
        for s in streams:
            with torch.cuda.stream(s):
                call()
    torch.cuda.synchronize()
    got = out.clone()
    out.zero_()
    call()
    torch.cuda.synchronize()
    assert torch.equal(got, out) and torch.any(out != 0)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.all(x == 1.0)
    model.close()
