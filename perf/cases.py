"""Performance cases: the calls that a variational Monte Carlo program makes, over the sizes it makes them at.

One optimisation step of a neural quantum state samples configurations from |psi|^2, evaluates their local
energies, and forms log-derivatives, forces and the stochastic-reconfiguration (SR) update.  Each case is one of
these calls (or a whole step, for the smallest network) on one of the library's networks, with seeded synthetic
weights and spins.  Sampling continues chains that the program keeps, as every step after the first does.

A case names its network (`arch`, lattice, `widths`), what is called (`kind`), how much of it, and the format.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2601_20782_amd as nqs
import workloads

DEV = "cuda:0"


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _case(name, kind, arch, dim, L, widths, **kw):
    c = {"kind": kind, "arch": arch, "dim": dim, "L": L, "widths": widths}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A whole SR step of the regularisation study's network (RBM on the 16-site chain, 1024 samples on 256
        # chains): small trainings run thousands of these, bound by latency and by the number of launches.
        _case("vmc_step_rbm_chain16", "vmc", "rbm", 1, 16, "16", chains=256, sweeps=4, burnin=2, dtype="bf16",
              shift=1e-2),
        # The headline sampler: RBM alpha = 2 on the 10 x 10 TFIM, 4096 chains, single flips.
        _case("sample_rbm_tfim10", "sample", "rbm", 2, 10, "200", chains=4096, sweeps=100, burnin=10, dtype="bf16",
              refresh=4),
        # Local energies of that run's samples (FP32 ratios) and their statistics.
        _case("eloc_rbm_tfim10", "eloc", "rbm", 2, 10, "200", n=409600, chains=4096, dtype="f32"),
        # Exchange sweeps of the two-layer network on the 10 x 10 Heisenberg lattice, 16384 chains.
        _case("sample_ffnn_heis10", "sample", "ffnn", 2, 10, "400,200", chains=16384, sweeps=20, burnin=0,
              dtype="bf16", refresh=4),
        # Its local energies in the sampling format, a sample count that fills no group or pass evenly.
        _case("eloc_ffnn_heis10", "eloc", "ffnn", 2, 10, "400,200", n=65001, chains=0, dtype="bf16"),
        # The largest network: one exchange sweep of 65536 chains of the three-layer network on the 20 x 20
        # lattice (batched forward passes).
        _case("sample_ffnn3_heis20", "sample", "ffnn", 2, 20, "1600,800,400", chains=65536, sweeps=1, burnin=0,
              dtype="bf16", refresh=0),
        # The residual convolutional network of the TFIM study: one sweep of 4096 chains in BF16.
        _case("sample_rescnn_tfim10", "sample", "rescnn", 2, 10, "16", blocks=4, chains=4096, sweeps=1, burnin=0,
              dtype="bf16", refresh=0),
        # Its local energies in the default format (a forward pass of every flipped configuration).
        _case("eloc_rescnn_tfim10", "eloc", "rescnn", 2, 10, "16", blocks=4, n=1000, chains=0, dtype="f32"),
        # log psi, the log-derivatives O of every sample (backward) and the forces, two-layer network.
        _case("grad_ffnn_heis10", "grad", "ffnn", 2, 10, "400,200", n=4001),
        # The SR step of that network around its solve: T from the samples, and the parameter update.
        _case("gram_update_ffnn_heis10", "gram_update", "ffnn", 2, 10, "400,200", n=6000),
        # The SR step of the headline RBM on one sweep's 4096 samples: T, the solve, the update.
        _case("sr_rbm_tfim10", "sr", "rbm", 2, 10, "200", n=4096, shift=1e-2, solver="cg"),
        # Energy of a complex-parameter RBM: sampling, then complex local energies of the samples; a chain
        # count that is no multiple of a workgroup's.
        _case("energy_crbm_tfim10", "energy", "crbm", 2, 10, "200", chains=3000, sweeps=10, burnin=2, dtype="f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, n):
    """n, or a size near it that is a multiple of nothing in particular."""
    return n if rng.random() < 0.4 else max(1, n - rng.randrange(max(1, n // 7)))


def draw(rng):
    kind = rng.choice(["vmc", "sample", "sample", "sample", "eloc", "eloc", "eloc", "grad", "gram_update", "sr",
                       "energy"])
    if kind == "vmc":
        L = rng.choice([8, 10, 12, 16, 20])
        return _case(None, kind, "rbm", 1, L, str(L * rng.choice([1, 2])), chains=_odd(rng, _log_int(rng, 32, 256)),
                     sweeps=4, burnin=rng.choice([1, 2, 5]), dtype=rng.choice(["bf16", "f16", "f32"]), shift=1e-2)
    if kind == "energy":
        L = rng.choice([4, 6, 8, 10])
        return _case(None, kind, "crbm", 2, L, str(L * L * rng.choice([1, 2])),
                     chains=_odd(rng, _log_int(rng, 256, 4096)), sweeps=rng.choice([4, 10, 20]),
                     burnin=rng.choice([0, 2]), dtype=rng.choice(["bf16", "f16", "f32"]))
    arch = rng.choice({"sample": ["rbm", "ffnn", "ffnn", "ffnn3", "rescnn"], "eloc": ["rbm", "ffnn", "ffnn", "rescnn"],
                       "grad": ["rbm", "ffnn", "ffnn"], "gram_update": ["ffnn", "ffnn3"], "sr": ["rbm"]}[kind])
    kw = {}
    if arch == "rbm":
        L = rng.choice([6, 8, 9, 10, 12, 14, 16] if kind == "eloc" else [6, 8, 9, 10, 12])
        N = L * L
        widths = [N * rng.choice([1, 2] if L > 10 else [1, 2, 3, 4])]
        flops = 6.0 * widths[0]                                # of one proposal or flip
    elif arch == "ffnn":
        L = rng.choice([4, 6, 8, 10])
        N = L * L
        w1 = min(400, _odd(rng, 4 * N))
        widths = [w1, max(8, min(200, _odd(rng, w1 // 2)))]
        flops = 2.0 * widths[0] * widths[1]
    elif arch == "ffnn3":
        arch, L = "ffnn", rng.choice([10, 12, 16, 20])
        N = L * L
        w1 = _odd(rng, 4 * N)
        widths = [w1, w1 // 2, w1 // 4]
        flops = 2.0 * (N * w1 + w1 * (w1 // 2) + (w1 // 2) * (w1 // 4))
    else:
        L = rng.choice([4, 6, 8, 10])
        N = L * L
        widths = [rng.choice([16, 32])]
        kw["blocks"] = rng.choice([2, 4])
        flops = 80.0 * N * kw["blocks"] * widths[0] * (widths[0] + 16)
    ws = ",".join(str(w) for w in widths)
    if kind == "sample":
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"] if len(widths) < 3 else ["bf16", "bf16", "f16", "e4m3"])
        slow = 12.0 if dtype == "f32" and arch == "ffnn" else 1.0
        chains = _odd(rng, _log_int(rng, 256, 16384))
        sweeps = rng.choice([1, 2, 5, 10, 20])
        cost = 1.0e12 if arch == "rbm" else 1.0e13
        sweeps = max(1, min(sweeps, int(cost / (chains * N * flops * slow))))
        chains = max(64, min(chains, int(cost / (sweeps * N * flops * slow))))
        return _case(None, kind, arch, 2, L, ws, chains=chains, sweeps=sweeps, burnin=0, dtype=dtype,
                     refresh=rng.choice([0, 1, 4]), **kw)
    if kind == "eloc":
        dtype = "f32" if arch in ("rbm", "rescnn") else rng.choice(["bf16", "f16", "f32"])
        slow = 20.0 if arch == "rescnn" else 10.0 if dtype == "f32" and arch == "ffnn" else 1.0
        n = _odd(rng, _log_int(rng, 1024, 300000))
        n = max(100, min(n, int((1.0e12 if arch == "rbm" else 1.0e13) / (N * flops * slow))))
        return _case(None, kind, arch, 2, L, ws, n=n, chains=0, dtype=dtype, **kw)
    P, prev = 0, N
    for w in widths:
        P, prev = P + w * (prev + 1), w
    if arch == "rbm":
        P += N
    if kind == "grad":
        return _case(None, kind, arch, 2, L, ws, n=min(_odd(rng, _log_int(rng, 500, 8000)), 480000000 // P))
    if kind == "gram_update":
        return _case(None, kind, arch, 2, L, ws, n=min(_odd(rng, _log_int(rng, 500, 8000)), 4000000000 // P))
    return _case(None, kind, arch, 2, L, ws, n=_odd(rng, _log_int(rng, 500, 5000)), shift=1e-2,
                 solver=rng.choice(["cg", "cg", "bf16", "f32"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _shape(case):
    L = int(case["L"])
    N = L if case["dim"] == 1 else L * L
    return L, N, [int(w) for w in str(case["widths"]).split(",")]


def _params(case, seed):
    _, N, widths = _shape(case)
    arch = case["arch"]
    if arch == "rbm":
        return workloads.rbm_params(N, widths[0], 0.1 if N <= 20 else 0.02, seed)
    if arch == "crbm":
        return workloads.crbm_params(N, widths[0], 0.02, 0.02, seed)
    if arch == "rescnn":
        return workloads.rescnn_params(widths[0], int(case["blocks"]), seed)
    return workloads.ffnn_params(N, widths, seed, 0.05)


def _exchange(case):
    """The dense networks run on the Heisenberg lattice, in its zero-magnetisation sector."""
    return case["arch"] == "ffnn"


def _model(case, params):
    L, N, widths = _shape(case)
    if case["arch"] == "rescnn":
        return nqs.Model.rescnn(L, widths[0], int(case["blocks"]), params)
    return nqs.Model(case["arch"], N, widths, params, marshall=_exchange(case), lat_dim=case["dim"], lat_L=L)


def _ham(case):
    L, N, _ = _shape(case)
    if _exchange(case):
        return nqs.Hamiltonian("heisenberg", case["dim"], L, 1.0, 0.0, True)
    return nqs.Hamiltonian("tfim", case["dim"], L, 1.0, -1.0 if case["dim"] == 1 else 3.04, True)


def _spins(case, n, gen):
    """Random configurations; zero magnetisation for exchange moves."""
    _, N, _ = _shape(case)
    if not _exchange(case):
        return (2 * torch.randint(0, 2, (n, N), generator=gen, device=DEV, dtype=torch.int8) - 1).contiguous()
    out = torch.empty(n, N, dtype=torch.int8, device=DEV)
    base = torch.ones(N, dtype=torch.int8, device=DEV)
    base[N // 2:] = -1
    for k in range(0, n, 65536):
        m = min(65536, n - k)
        out[k:k + m] = base[torch.rand(m, N, generator=gen, device=DEV).argsort(dim=1)]
    return out


def _inputs(case, seed):
    """Parameters, and the generator that every other input is drawn from."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1000003 * seed + 17)
    return _params(case, seed), gen


def prepare(case, seed):
    params, gen = _inputs(case, seed)
    _, N, _ = _shape(case)
    kind = case["kind"]
    st = {"case": case, "model": _model(case, params), "ham": _ham(case)}
    f64 = dict(dtype=torch.float64, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    P = st["model"].n_params
    if kind in ("sample", "energy", "vmc"):
        C, S = case["chains"], case["sweeps"]
        st["cfg"] = nqs.SampleConfig(n_chains=C, n_sweeps=S, n_burnin=case["burnin"], seed=seed, dtype=case["dtype"],
                                     move="exchange" if _exchange(case) else "flip", init_chains=False,
                                     refresh_sweeps=case.get("refresh", 0))
        st["chains"] = _spins(case, C, gen)
        st["samples"] = torch.empty(S, C, N, dtype=torch.int8, device=DEV)
        st["accepted"] = torch.empty(C, dtype=torch.int64, device=DEV)
        st["model"].prepare(case["dtype"])
        n = S * C
    else:
        n = case["n"]
        st["samples"] = _spins(case, n, gen)
    if kind in ("eloc", "energy", "vmc"):
        st["eloc"] = torch.empty(n, **f64)
        st["eloc_im"] = torch.empty(n, **f64) if case["arch"] == "crbm" else None
        st["stats"] = torch.empty(4, **f64)
    elif kind in ("grad", "sr", "gram_update"):
        st["eloc"] = 3.0 * torch.randn(n, generator=gen, **f64) - 100.0
    if kind == "eloc":
        st["model"].prepare(case["dtype"])
    if kind == "grad":
        st["logpsi"], st["O"] = torch.empty(n, **f32), torch.empty(n, P, **f32)
        st["F"] = torch.empty(P, **f64)
    if kind in ("sr", "gram_update", "vmc"):
        st["T"] = torch.empty(n, n, **f32)
        st["y"] = torch.empty(n, **f64)
        st["master"] = torch.from_numpy(params).to(DEV)
    if kind == "gram_update":
        st["y"] = torch.randn(n, generator=gen, **f64)
    if kind in ("grad", "sr", "gram_update", "vmc"):
        st["model"].prepare("f32")
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _sample(st):
    case, cfg = st["case"], st["cfg"]
    _, N, _ = _shape(case)
    nqs.nqs_sample(st["model"], cfg, st["chains"], st["samples"], None, st["accepted"])
    cfg.step_offset += (cfg.n_burnin + cfg.n_sweeps) * N   # the next pass goes on with the chains' random streams


def _solve(st, T, eps, y):
    solver = st["case"].get("solver", "cg")
    if solver == "cg":
        nqs.nqs_sr_solve(T, eps, st["case"]["shift"], y, tol=1e-12, max_iter=2000)
    else:
        nqs.nqs_sr_solve_mixed(T, eps, st["case"]["shift"], y, solver, tol=1e-12, max_iter=2000)


def run(st):
    case, model = st["case"], st["model"]
    kind = case["kind"]
    _, N, _ = _shape(case)
    if kind == "sample":
        _sample(st)
        return {"samples": st["samples"], "chains": st["chains"], "accepted": st["accepted"]}
    if kind == "energy":
        _sample(st)
        flat = st["samples"].view(-1, N)
        nqs.nqs_local_energy_complex(model, st["ham"], flat, st["eloc"], st["eloc_im"], case["dtype"])
        nqs.nqs_energy_stats(st["eloc"], case["chains"], st["stats"])
        return {"samples": st["samples"], "accepted": st["accepted"], "re": st["eloc"], "im": st["eloc_im"],
                "stats": st["stats"]}
    if kind == "eloc":
        nqs.nqs_local_energy(model, st["ham"], st["samples"], st["eloc"], case["dtype"])
        nqs.nqs_energy_stats(st["eloc"], case["chains"], st["stats"])
        return {"eloc": st["eloc"], "energy": st["stats"][:2] if case["chains"] == 0 else st["stats"]}
    if kind == "grad":
        nqs.nqs_logpsi_grad(model, st["samples"], logpsi=st["logpsi"], O=st["O"])
        nqs.nqs_forces(st["O"], st["eloc"], st["F"])
        return {"logpsi": st["logpsi"], "O": st["O"], "F": st["F"]}
    if kind == "gram_update":
        nqs.nqs_sample_gram_factored(model, st["samples"], st["T"])
        new = st["master"].clone()
        nqs.nqs_sr_update(model, st["samples"], st["y"], 0.01, new)
        return {"T": st["T"], "params": new}
    if kind == "sr":
        nqs.nqs_sample_gram_factored(model, st["samples"], st["T"])
        _solve(st, st["T"], st["eloc"], st["y"])
        new = st["master"].clone()
        nqs.nqs_sr_update(model, st["samples"], st["y"], 0.01, new)
        return {"T": st["T"], "y": st["y"], "params": new}
    # vmc: one optimisation step from the parameters in hand
    model.set_params_device(st["master"])
    model.prepare(case["dtype"])
    _sample(st)
    flat = st["samples"].view(-1, N)
    nqs.nqs_local_energy(model, st["ham"], flat, st["eloc"])
    nqs.nqs_energy_stats(st["eloc"], case["chains"], st["stats"])
    nqs.nqs_sample_gram_factored(model, flat, st["T"])
    _solve(st, st["T"], st["eloc"], st["y"])
    new = st["master"].clone()
    nqs.nqs_sr_update(model, flat, st["y"], 0.05, new)
    return {"samples": st["samples"], "accepted": st["accepted"], "eloc": st["eloc"], "stats": st["stats"],
            "T": st["T"], "y": st["y"], "params": new}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _forward_flops(case):
    _, N, widths = _shape(case)
    if case["arch"] == "rescnn":
        return 18.0 * N * widths[0] * (1 + 2 * int(case["blocks"]) * widths[0])
    if case["arch"] in ("rbm", "crbm"):
        return 2.0 * N * widths[0] * (4 if case["arch"] == "crbm" else 1)
    dims = [N] + widths
    return 2.0 * sum(a * b for a, b in zip(dims, dims[1:]))


def _ratio_flops(case):
    """One amplitude ratio of a flip or an exchange.  The product forms of the RBMs need 4 (complex: 20) operations
    per hidden unit; a two-layer network updates its first layer and multiplies the second; the others run a
    forward pass."""
    _, N, widths = _shape(case)
    if case["arch"] in ("rbm", "crbm"):
        return (20.0 if case["arch"] == "crbm" else 4.0) * widths[0]
    if case["arch"] == "ffnn" and len(widths) == 2:
        return 4.0 * widths[0] + 2.0 * widths[0] * widths[1]
    return _forward_flops(case)


def _n_params(case):
    _, N, widths = _shape(case)
    if case["arch"] == "rescnn":
        F, R = widths[0], int(case["blocks"])
        return 10 * F + R * (2 * F + 2 * (9 * F * F + F)) + 2 * F
    dims = [N] + widths
    P = sum(b * (a + 1) for a, b in zip(dims, dims[1:]))
    return P + (N if case["arch"] == "rbm" else 2 * N + P if case["arch"] == "crbm" else 0)


def work(case):
    _, N, widths = _shape(case)
    kind, P = case["kind"], _n_params(case)
    nbytes, flops = 4.0 * P, 0.0
    # half of the exchanges swap equal spins; every site has two bonds, half of them between unequal spins
    share = 0.5 if _exchange(case) else 1.0
    if kind in ("sample", "energy", "vmc"):
        C, S = case["chains"], case["sweeps"]
        n = C * S
        flops += C * (S + case["burnin"]) * N * share * _ratio_flops(case)
        nbytes += N * (n + 2 * C) + 8 * C
    else:
        n = case["n"]
    if kind in ("eloc", "energy", "vmc"):
        flops += n * N * _ratio_flops(case) * (case["dim"] * share if _exchange(case) else 1.0)
        nbytes += n * (N + (16 if case["arch"] == "crbm" else 8))
    if kind == "grad":
        flops += 4.0 * n * P
        nbytes += n * N + 2 * 4.0 * n * P                      # O is written, and read by the forces
    if kind in ("sr", "gram_update", "vmc"):
        dims = [N] + widths
        factors = sum(dims[:-1]) + sum(widths)
        flops += n * n * float(factors) + 6.0 * n * P          # the upper triangle of T; forward, backward, update
        nbytes += n * N + 4.0 * n * n
    if kind in ("sr", "vmc"):
        nbytes += 4.0 * n * n                                  # the solve reads T (once, at the least)
        flops += 2.0 * n * n
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _round(x, dtype):
    """FP64 values rounded to a format, in FP64."""
    if dtype == "bf16":
        return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)
    if dtype == "f16":
        return x.to(torch.float16).to(torch.float64)
    return x.to(torch.float32).to(torch.float64) if dtype == "f32" else x


def _logcosh(z):
    a = z.abs()
    return a + torch.log1p(torch.exp(-2.0 * a)) - math.log(2.0)


def _dense_layers(case, params, dtype):
    _, N, widths = _shape(case)
    p = _round(torch.from_numpy(params).to(DEV), dtype)
    out, off, prev = [], 0, N
    for w in widths:
        out.append((p[off:off + w * prev].view(w, prev), p[off + w * prev:off + w * (prev + 1)]))
        off, prev = off + w * (prev + 1), w
    return out


def _logpsi_fn(case, params, dtype):
    """log |psi| of FP64 configurations [n][N], the operands of every product in the format."""
    L, N, widths = _shape(case)
    if case["arch"] == "rbm":
        p = _round(torch.from_numpy(params).to(DEV), dtype)
        M = widths[0]
        a, b, W = p[:N], p[N:N + M], p[N + M:].view(M, N)
        return lambda s: s @ a + _logcosh(s @ W.T + b).sum(dim=1)
    if case["arch"] == "ffnn":
        layers = _dense_layers(case, params, dtype)

        def dense(s):
            h = s
            for l, (W, b) in enumerate(layers):
                h = h @ W.T + b
                if l + 1 < len(layers):
                    h = _round(torch.relu(h), dtype)
            return _logcosh(h).sum(dim=1)
        return dense
    F, R = widths[0], int(case["blocks"])
    p = _round(torch.from_numpy(params).to(DEV), dtype)
    off = 0

    def take(*shape):
        nonlocal off
        n = math.prod(shape)
        off += n
        return p[off - n:off].view(*shape)

    w0, b0 = take(F, 1, 9), take(F)
    blocks = [(take(F), take(F), take(F, F, 9), take(F), take(F, F, 9), take(F)) for _ in range(R)]
    gf, bf = take(F), take(F)
    site = torch.arange(N, device=DEV)
    x, y = site // L, site % L
    nbr = torch.stack([((x + k // 3 - 1) % L) * L + (y + k % 3 - 1) % L for k in range(9)])   # [9][N]

    def conv(h, W, b):           # h [n][N][C]
        n, C = h.shape[0], h.shape[2]
        cols = h[:, nbr.T.reshape(-1), :].view(n, N, 9 * C)
        return cols @ W.permute(2, 1, 0).reshape(9 * C, -1) + b

    def ln(h, g, be):
        mu = h.mean(dim=2, keepdim=True)
        var = ((h - mu) ** 2).mean(dim=2, keepdim=True)
        return (h - mu) / torch.sqrt(var + 1e-6) * g + be

    def gelu(z):
        return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))

    def net(s):
        h = conv(s.unsqueeze(2), w0, b0)
        for g, be, w1, b1, w2, b2 in blocks:
            t = _round(gelu(ln(h, g, be)), dtype)
            h = h + conv(_round(gelu(conv(t, w1, b1)), dtype), w2, b2)
        return ln(h, gf, bf).sum(dim=(1, 2))
    return net


def _exact_eloc(case, params, samples):
    L, N, widths = _shape(case)
    f = _logpsi_fn(case, params, case["dtype"])
    site = torch.arange(N, device=DEV)
    if case["dim"] == 1:
        bonds = torch.stack([site, (site + 1) % L], dim=1)
    else:
        x, y = site // L, site % L
        bonds = torch.cat([torch.stack([site, ((x + 1) % L) * L + y], dim=1),
                           torch.stack([site, x * L + (y + 1) % L], dim=1)])
    rows = 2 * N + 1
    width = {"rescnn": 9 * N * widths[0] * 2, "rbm": 2 * widths[0]}.get(case["arch"], 2 * max(widths))
    chunk = max(1, int(4e8 / (rows * width)))
    out = torch.empty(samples.shape[0], dtype=torch.float64, device=DEV)
    for k in range(0, samples.shape[0], chunk):
        s = samples[k:k + chunk].double()
        n = s.shape[0]
        diag = (s[:, bonds[:, 0]] * s[:, bonds[:, 1]]).sum(dim=1)
        f0 = f(s)
        if _exchange(case):
            # 2 psi(s') / psi(s) for every antiparallel bond; nearest neighbours lie on different sublattices, so
            # the Marshall sign of the swap is -1
            s2 = s.unsqueeze(1).repeat(1, bonds.shape[0], 1)
            q = torch.arange(bonds.shape[0], device=DEV)
            s2[:, q, bonds[:, 0]], s2[:, q, bonds[:, 1]] = s[:, bonds[:, 1]], s[:, bonds[:, 0]]
            anti = (s[:, bonds[:, 0]] != s[:, bonds[:, 1]])
            r = torch.zeros(n, bonds.shape[0], dtype=torch.float64, device=DEV)
            r[anti] = torch.exp(f(s2[anti]) - f0.unsqueeze(1).expand_as(r)[anti])
            out[k:k + chunk] = diag - 2.0 * r.sum(dim=1)
        else:
            flips = s.unsqueeze(1) * (1.0 - 2.0 * torch.eye(N, dtype=torch.float64, device=DEV))
            r = torch.exp(f(flips.reshape(-1, N)).view(n, N) - f0.unsqueeze(1))
            out[k:k + chunk] = diag + (-1.0 if case["dim"] == 1 else 3.04) * r.sum(dim=1)
    return out


def _factors(case, params, samples):
    """Per layer (delta, input) with O_W = delta x input, O_b = delta, from the FP32-rounded parameters."""
    _, N, widths = _shape(case)
    s = samples.double()
    if case["arch"] == "rbm":
        p = _round(torch.from_numpy(params).to(DEV), "f32")
        M = widths[0]
        theta = s @ p[N + M:].view(M, N).T + p[N:N + M]
        return [(torch.tanh(theta), s)], s @ p[:N] + _logcosh(theta).sum(dim=1)
    layers = _dense_layers(case, params, "f32")
    ins, zs, h = [], [], s
    for l, (W, b) in enumerate(layers):
        ins.append(h)
        z = h @ W.T + b
        zs.append(z)
        h = torch.relu(z)
    d = torch.tanh(zs[-1])
    fac = [None] * len(layers)
    for l in range(len(layers) - 1, -1, -1):
        fac[l] = (d, ins[l])
        if l:
            d = (d @ layers[l][0]) * (zs[l - 1] > 0)
    return fac, _logcosh(zs[-1]).sum(dim=1)


def _exact_O(case, fac):
    n = fac[0][0].shape[0]
    cols = [fac[0][1]] if case["arch"] == "rbm" else []
    for d, h in fac:
        ow = torch.bmm(d.unsqueeze(2), h.unsqueeze(1)).view(n, -1)
        cols += [d, ow] if case["arch"] == "rbm" else [ow, d]
    return torch.cat(cols, dim=1)


def _exact_T(case, fac):
    n = fac[0][0].shape[0]
    K = torch.zeros(n, n, dtype=torch.float64, device=DEV)
    for d, h in fac:
        K += (d @ d.T) * (h @ h.T + 1.0)
    if case["arch"] == "rbm":
        K += fac[0][1] @ fac[0][1].T
    return (K - K.mean(dim=0, keepdim=True) - K.mean(dim=1, keepdim=True) + K.mean()) / n


def _exact_update(case, params, fac, y, lr):
    g = (y - y.mean()) / y.numel()
    parts = [fac[0][1].T @ g] if case["arch"] == "rbm" else []
    for d, h in fac:
        gd = d * g.unsqueeze(1)
        ow = (gd.T @ h).reshape(-1)
        parts += [gd.sum(dim=0), ow] if case["arch"] == "rbm" else [ow, gd.sum(dim=0)]
    return torch.from_numpy(params).to(DEV) - lr * torch.cat(parts)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sample", "energy", "vmc"):
        return None                      # whole numbers, and values of the samples that they are
    params, gen = _inputs(case, seed)
    n = case["n"]
    samples = _spins(case, n, gen)
    if kind == "eloc":
        e = _exact_eloc(case, params, samples)
        stats = [e.mean(), e.var()]
        if case["chains"]:
            cm = e.view(-1, case["chains"]).mean(dim=0)
            stats += [cm.std() / math.sqrt(case["chains"]), torch.tensor(float(n), dtype=torch.float64, device=DEV)]
        return {"eloc": e, "energy": torch.stack(stats)}
    eps = 3.0 * torch.randn(n, generator=gen, dtype=torch.float64, device=DEV) - 100.0
    fac, logpsi = _factors(case, params, samples)
    if kind == "grad":
        O = _exact_O(case, fac)
        F = (O.T @ eps) / n - O.mean(dim=0) * eps.mean()
        return {"logpsi": logpsi, "O": O, "F": F}
    T = _exact_T(case, fac)
    if kind == "gram_update":
        y = torch.randn(n, generator=gen, dtype=torch.float64, device=DEV)
        return {"T": T, "params": _exact_update(case, params, fac, y, 0.01)}
    A = T.clone()
    A.diagonal().add_(case["shift"])
    y = torch.cholesky_solve((eps - eps.mean()).unsqueeze(1), torch.linalg.cholesky(A)).squeeze(1)
    return {"T": T, "y": y, "params": _exact_update(case, params, fac, y, 0.01)}
