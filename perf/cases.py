"""Performance cases of the block-wise ALIF library on one MI355X.

Each case is one call, or one short chain of calls, that a program using the
library makes: a layer's forward (and backward) on injected current or on
presynaptic spikes, a recurrent layer, the neural-fit epoch, a classifier's
training step through torch.autograd, the Eq. 3 projections on their own, the
device-drawn OU current and a burst of serving requests. ``listed()`` gives the
named cases, ``draw(rng)`` further ones over the same ranges of sizes.

Times of a case cover the whole chain through the public entry points. Inputs
come from torch generators seeded by ``seed`` (Poisson / Bernoulli spikes, OU
currents, Normal(0, 1/sqrt(fan_in)) weights, uniform time constants), so they do
not depend on the library. ``exact`` repeats a case in 64 bits with plain torch
operations, step by step (the standard model, Eqs. 1-5 of the paper, and its
detached surrogate adjoint).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2311_11390_amd import _lib as L
from paper_2311_11390_amd import alif, serving

DEV = "cuda"
TAU_VR = 100.0    # van Rossum time constant of the fits (ms)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _layer(**kw):
    c = dict(kind="layer", batch=1, T=1000, n_in=0, n=100, tr=2, dt=1.0, gemm="fp32", density=0.02,
             train=False, dx=False, traces=False)
    c.update(kw)
    return c


def listed():
    return [
        # inference on one sample of the synthetic spike dataset: 200 -> 100, batch 1, the smallest
        # layer in use; 500 blocks in sequence, so latency and launches count
        _layer(name="single_layer_forward", T=1000, n_in=200, n=100, tr=2, density=0.02),
        # the fine-DT fit: injected current, 64 x 256 neurons, DT 0.05 ms, ARP 2 ms, gradients of the
        # neuron parameters only (the largest step in use)
        _layer(name="fine_dt_fit", batch=64, T=20000, n=256, tr=40, dt=0.05, train=True),
        # one layer of the speed benchmark with a long refractory period that no segment split fills
        # (T_R 100): 200 -> 256, FP32 GEMMs, Poisson input up to 200 Hz
        _layer(name="speed_layer_long_blocks", batch=64, T=2048, n_in=200, n=256, tr=100, density=0.1, train=True),
        # a hidden layer of the speed benchmark's deeper networks: 512 -> 512, FP32, with the gradient
        # passed to the layer below
        _layer(name="hidden_layer_fp32", batch=64, T=1024, n_in=512, n=512, tr=40, density=0.02, train=True, dx=True),
        # the hidden layer of the three-layer BF16 network: 1024 -> 1024, batch 128, T 2000, T_R 4,
        # driven by another layer's sparse spikes
        _layer(name="hidden_layer_bf16", batch=128, T=2000, n_in=1024, n=1024, tr=4, dt=0.5, gemm="bf16",
               density=0.002, train=True, dx=True),
        # a BF16 layer on denser input (50 Hz at 1 ms), where the projections stay dense GEMMs
        _layer(name="input_layer_bf16_dense", batch=64, T=1000, n_in=700, n=1024, tr=2, gemm="bf16", density=0.05,
               train=True, dx=True),
        # one training step of the SHD-shaped classifier through torch.autograd: 700 -> 512 ALIF -> 20
        # leaky readout, cross-entropy; returns the logits and every gradient
        dict(name="classifier_step", kind="classifier", batch=32, T=1000, n_in=700, n=512, classes=20, tr=2, dt=1.0,
             density=0.025),
        # the recurrent layer at the fine-DT shape, forward and backward with the recurrent weights' gradient
        dict(name="recurrent_fine_dt", kind="recurrent", batch=64, T=20000, n=256, tr=40, dt=0.05),
        # one epoch of the neural fits: forward, van Rossum loss against four repeats, backward, Adam
        dict(name="fit_epoch", kind="fit", batch=4, repeats=4, T=20000, n=2048, tr=20, dt=0.1),
        # the Eq. 3 projection and its two gradients on their own (FP32 GEMMs), as a program that
        # composes its own layer calls them
        dict(name="projections_fp32", kind="project", batch=32, T=1000, n_in=700, n=512, gemm="fp32", x="u8",
             density=0.025),
        # an injected OU current drawn on the device: one stimulus of the neural fits (2048 neurons, 2 s)
        dict(name="ou_current", kind="ou", T=20000, n=2048, dt=0.1),
        # a burst of eight uneven serving requests answered with spike events
        dict(name="serving_burst", kind="serve", requests=8, t_max=20000, n_max=1024, sizes=7),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["current", "current", "spikes", "spikes", "spikes", "classifier", "recurrent", "fit", "project",
                       "project", "ou", "serve"])
    tr = rng.choice([2, 3, 4, 5, 7, 10, 16, 20, 23, 31, 40, 47, 64, 80, 100, 120])
    if kind == "current":      # fits and simulations on injected current
        n = _log_int(rng, 20, 2048)
        T = _log_int(rng, 500, 20000)
        b = max(1, min(_log_int(rng, 1, 128), int(2e8 // (n * T))))
        return _layer(batch=b, T=T, n=n, tr=tr, dt=2.0 / tr, train=rng.random() < 0.7, traces=rng.random() < 0.2)
    if kind == "spikes":       # network layers
        n = _log_int(rng, 20, 1024)
        n_in = rng.choice([200, 700, _log_int(rng, 20, 1024)])
        T = _log_int(rng, 250, 2048)
        b = max(1, min(_log_int(rng, 1, 128), int(6.5e7 // (max(n, n_in) * T))))
        train = rng.random() < 0.75
        return _layer(batch=b, T=T, n_in=n_in, n=n, tr=tr, dt=1.0, gemm=rng.choice(["fp32", "fp32", "bf16"]),
                      density=math.exp(rng.uniform(math.log(0.002), math.log(0.1))), train=train,
                      dx=train and rng.random() < 0.5)
    if kind == "classifier":
        return dict(kind="classifier", batch=_log_int(rng, 8, 64), T=_log_int(rng, 250, 1500), n_in=700,
                    n=_log_int(rng, 64, 512), classes=rng.choice([10, 20, 35]), tr=rng.choice([2, 4, 5, 10]), dt=1.0,
                    density=rng.uniform(0.01, 0.05))
    if kind == "recurrent":
        n = _log_int(rng, 32, 256)
        T = _log_int(rng, 1000, 15000)
        return dict(kind="recurrent", batch=max(1, min(_log_int(rng, 8, 64), int(2e8 // (n * T)))), T=T, n=n,
                    tr=rng.choice([10, 20, 40, 47, 64]), dt=0.05)
    if kind == "fit":
        return dict(kind="fit", batch=rng.choice([2, 4, 8]), repeats=rng.choice([1, 3, 4]), T=_log_int(rng, 500, 15000),
                    n=_log_int(rng, 256, 1024), tr=rng.choice([2, 4, 10, 20, 40, 80]), dt=0.1)
    if kind == "project":
        return dict(kind="project", batch=_log_int(rng, 4, 64), T=_log_int(rng, 250, 2000),
                    n_in=rng.choice([200, 512, 700, _log_int(rng, 32, 1024)]), n=_log_int(rng, 20, 1024),
                    gemm=rng.choice(["fp32", "fp32", "bf16"]), x=rng.choice(["u8", "u8", "bf16", "f32"]),
                    density=math.exp(rng.uniform(math.log(0.002), math.log(0.1))))
    if kind == "ou":
        return dict(kind="ou", T=_log_int(rng, 500, 30000), n=_log_int(rng, 64, 1024), dt=rng.choice([0.05, 0.1, 1.0]))
    return dict(kind="serve", requests=rng.randint(1, 8), t_max=_log_int(rng, 2000, 20000),
                n_max=_log_int(rng, 128, 1024), sizes=rng.randint(0, 10**6))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device=DEV) * (hi - lo) + lo


def _ou(g, B, T, N, dt, tau, mean, sd):
    """OU process [B][T][N], exact discretisation, float32."""
    e = math.exp(-dt / tau)
    x = torch.randn(B, T, N, generator=g, device=DEV).mul_(sd * math.sqrt(1.0 - e * e))
    x[:, 0].div_(math.sqrt(1.0 - e * e))
    k = 1                      # inclusive scan by doubling, out to where e^k is negligible
    while k < T and e ** k > 1e-9:
        x[:, k:] = x[:, k:] + (e ** k) * x[:, :-k]
        k *= 2
    return x.add_(mean).contiguous()


def _spikes(g, B, T, n, density, dtype=torch.uint8):
    """Bernoulli spikes [B][T][n], a rate per channel (uniform, mean ``density``)."""
    rate = _uniform(g, 0.0, 2.0 * density, n)
    return (torch.rand(B, T, n, generator=g, device=DEV) < rate).to(dtype)


def _params(g, n, bias):
    return {"tau_mem": _uniform(g, 10.0, 30.0, n), "tau_adapt": _uniform(g, 100.0, 300.0, n),
            "d": torch.full((n,), 1.8, device=DEV), "theta0": torch.ones(n, device=DEV),
            "bias": _uniform(g, 1.0, 2.0, n) if bias else None}


def _weights(g, n_out, n_in):
    return torch.randn(n_out, n_in, generator=g, device=DEV) / math.sqrt(n_in)


def _layer_inputs(case, seed):
    g = _gen(seed)
    B, T, n, n_in = case["batch"], case["T"], case["n"], case["n_in"]
    s = {"p": _params(g, n, bias=n_in > 0)}
    if n_in:
        s["inp"], s["W"] = _spikes(g, B, T, n_in, case["density"]), _weights(g, n, n_in)
    else:
        s["inp"], s["W"] = _ou(g, B, T, n, case["dt"], 5.0, 0.8, 0.5), None
    if case["train"]:
        if n_in:    # dL/dS of a layer below another one: dense, zero mean
            s["gs"] = torch.randn(B, T, n, generator=g, device=DEV).mul_(1e-3)
        else:       # gradient of a smoothed train difference: slow in time
            s["gs"] = _ou(g, B, T, n, case["dt"], 2.0, 0.0, 1e-3)
    return s


def _classifier_inputs(case, seed):
    g = _gen(seed)
    B, T, n, C = case["batch"], case["T"], case["n"], case["classes"]
    return {"x": _spikes(g, B, T, case["n_in"], case["density"]), "W": _weights(g, n, case["n_in"]),
            "p": _params(g, n, bias=True), "Wr": _weights(g, C, n), "tr": torch.full((C,), 20.0, device=DEV),
            "labels": torch.randint(0, C, (B,), generator=g, device=DEV)}


def _recurrent_inputs(case, seed):
    g = _gen(seed)
    B, T, n = case["batch"], case["T"], case["n"]
    return {"inp": _ou(g, B, T, n, case["dt"], 5.0, 0.8, 0.5), "p": _params(g, n, bias=False),
            "Wrec": 0.5 * _weights(g, n, n), "gs": _ou(g, B, T, n, case["dt"], 2.0, 0.0, 1e-3)}


FIT = (("tau_mem", 0.5, 1.0, 200.0), ("tau_adapt", 5.0, 5.0, 2000.0), ("d", 0.01, 0.0, 5.0),
       ("theta0", 0.01, 0.05, 10.0), ("bias", 0.01, -5.0, 5.0))    # parameter, learning rate, bounds


def _fit_inputs(case, seed):
    g = _gen(seed)
    B, R, T, n = case["batch"], case["repeats"], case["T"], case["n"]
    p = {"tau_mem": _uniform(g, 15.0, 25.0, n), "tau_adapt": _uniform(g, 80.0, 120.0, n),
         "d": _uniform(g, 0.08, 0.12, n), "theta0": _uniform(g, 0.9, 1.1, n), "bias": _uniform(g, -0.05, 0.05, n)}
    rate = 15.0 * case["dt"] * 1e-3      # the recorded trains fire at about 15 Hz
    tgt = torch.empty(B, R, T, n, dtype=torch.uint8, device=DEV)
    for b in range(B):
        tgt[b] = torch.rand(R, T, n, generator=g, device=DEV) < rate
    return {"inp": _ou(g, B, T, n, case["dt"], 5.0, 1.2, 0.5), "targets": tgt, "p": p}


_XDT = {"u8": torch.uint8, "bf16": torch.bfloat16, "f32": torch.float32}


def _project_inputs(case, seed):
    g = _gen(seed)
    B, T, n, n_in = case["batch"], case["T"], case["n"], case["n_in"]
    return {"x": _spikes(g, B, T, n_in, case["density"], _XDT[case["x"]]), "W": _weights(g, n, n_in),
            "bias": _uniform(g, 1.0, 2.0, n), "gI": torch.randn(B, T, n, generator=g, device=DEV).mul_(1e-3)}


def _serve_sizes(case):
    """(N, T, DT) of each request, like the serving stream's: N and T uniform, DT in {1, 0.1, 0.05} ms."""
    g = np.random.Generator(np.random.PCG64(case["sizes"]))
    return [(int(g.integers(64, case["n_max"] + 1)), int(g.integers(500, case["t_max"] + 1)),
             float(g.choice([1.0, 0.1, 0.05]))) for _ in range(case["requests"])]


def _serve_requests(case, seed):
    """ARP 2 ms, an OU current drawn on the device, answered with spike events."""
    g = np.random.Generator(np.random.PCG64(seed))
    return [serving.Request(
        T=T, dt=dt, arp=2.0, tau_mem=g.uniform(10, 30, N).astype(np.float32),
        tau_adapt=g.uniform(100, 300, N).astype(np.float32), d=np.full(N, 1.8, np.float32),
        theta0=np.ones(N, np.float32), seed=int(g.integers(1, 2**62)), want_spikes=False,
        events_capacity=N * (2 + int(T * dt * 0.02)))     # room for 20 Hz
        for N, T, dt in _serve_sizes(case)]


def _alif_params(p):
    return alif.Params(p["tau_mem"], p["tau_adapt"], p["d"], p["theta0"], p["bias"])


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "layer":
        st.update(_layer_inputs(case, seed))
        st["P"] = _alif_params(st["p"])
    elif kind == "classifier":
        st.update(_classifier_inputs(case, seed))
        for t in (st["W"], st["Wr"], st["tr"], *st["p"].values()):
            t.requires_grad_()
    elif kind == "recurrent":
        st.update(_recurrent_inputs(case, seed))
        st["P"] = _alif_params(st["p"])
    elif kind == "fit":
        st.update(_fit_inputs(case, seed))
        B, R, T, n = case["batch"], case["repeats"], case["T"], case["n"]
        # what a fitting program keeps from epoch to epoch: optimiser state and loss buffers
        st["m"] = {k: torch.zeros(n, device=DEV) for k, *_ in FIT}
        st["v"] = {k: torch.zeros(n, device=DEV) for k, *_ in FIT}
        st["ws"] = alif.van_rossum_workspace(B, R, T, n, DEV)
    elif kind == "project":
        st.update(_project_inputs(case, seed))
    elif kind == "serve":
        st["requests"] = _serve_requests(case, seed)
        st["server"] = serving.Server(8 << 30, max_slots=8)
    else:
        st["seed"] = seed
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

_GEMM = {"fp32": L.GEMM_FP32, "bf16": L.GEMM_BF16}
_GRADS = ("grad_tau_mem", "grad_tau_adapt", "grad_d", "grad_theta0", "grad_bias")


def run(st):
    return _RUN[st["case"]["kind"]](st, st["case"])


def _run_layer(st, c):
    f = alif.forward(st["inp"], st["P"], c["dt"], c["dt"] * c["tr"], st["W"], gemm_precision=_GEMM[c["gemm"]],
                     want_v=c["traces"], want_theta=c["traces"], save=c["train"])
    out = {"spikes": f["spikes"]}
    if c["traces"]:
        out.update(v=f["v"], theta=f["theta"])
    if c["train"]:
        g = alif.backward(f, st["inp"], st["P"], st["W"], grad_spikes=st["gs"], want_grad_W=st["W"] is not None,
                          want_grad_input=c["dx"])
        out.update({k: g[k] for k in _GRADS})
        if st["W"] is not None:
            out["grad_W"] = g["grad_W"]
        if c["dx"]:
            out["grad_input"] = g["grad_input"]
    return out


def _run_classifier(st, c):
    p = st["p"]
    S, _, _ = alif.BlockALIF.apply(st["x"], st["W"], p["tau_mem"], p["tau_adapt"], p["d"], p["theta0"], p["bias"],
                                   {"dt": c["dt"], "arp": c["dt"] * c["tr"]})
    logits = alif.Readout.apply(S, st["Wr"], st["tr"], c["dt"])
    loss = torch.nn.functional.cross_entropy(logits, st["labels"])
    leaves = [st["W"], st["Wr"], st["tr"], *p.values()]
    grads = torch.autograd.grad(loss, leaves)
    return {"logits": logits.detach(), "loss": loss.detach(), "grads": list(grads)}


def _run_recurrent(st, c):
    f = alif.forward_recurrent(st["inp"], st["P"], c["dt"], c["dt"] * c["tr"], st["Wrec"])
    g = alif.backward_recurrent(f, st["inp"], st["P"], grad_spikes=st["gs"])
    return {"spikes": f["spikes"], "current": f["current"], "grad_W_rec": g["grad_W_rec"],
            **{k: g[k] for k in _GRADS}}


def _run_fit(st, c):
    # the epoch updates copies of the parameters and of Adam's state, so that a pass can be repeated
    p = {k: t.clone() for k, t in st["p"].items()}
    m = {k: t.clone() for k, t in st["m"].items()}
    v = {k: t.clone() for k, t in st["v"].items()}
    P = _alif_params(p)
    f = alif.forward(st["inp"], P, c["dt"], c["dt"] * c["tr"], save=True)
    dist, grad, _ = alif.van_rossum(f["spikes"], st["targets"], c["dt"], TAU_VR,
                                    scale=1.0 / (c["batch"] * c["repeats"]), workspace=st["ws"])
    g = alif.backward(f, st["inp"], P, grad_spikes=grad)
    for k, lr, lo, hi in FIT:
        alif.adam_step(p[k], g["grad_" + k], m[k], v[k], 1, lr, lo=lo, hi=hi)
    return {"spikes": f["spikes"], "dist": dist, "grad_spikes": grad, **{k: g[k] for k in _GRADS},
            "params": p, "m": m, "v": v}


def _run_project(st, c):
    gp = _GEMM[c["gemm"]]
    kind = {"u8": L.INPUT_SPIKES_U8, "bf16": L.INPUT_SPIKES_BF16, "f32": L.INPUT_SPIKES_F32}[c["x"]]
    return {"current": alif.input_current(st["x"], st["W"], st["bias"], gemm_precision=gp),
            "grad_W": alif.weight_grad(st["gI"], st["x"], gemm_precision=gp),
            "grad_input": alif.input_grad(st["gI"], st["W"], kind, gemm_precision=gp)}


def _run_ou(st, c):
    return alif.ou_current(c["T"], c["n"], c["dt"], 5.0, 0.8, 0.5, seed=st["seed"])


def _run_serve(st, c):
    tickets = [st["server"].submit(r) for r in st["requests"]]
    out = np.zeros((len(tickets), max(r.events_capacity for r in st["requests"])), np.uint32)   # a row a request
    counts = np.zeros(len(tickets), np.int64)
    for i, t in enumerate(tickets):
        r = st["server"].wait(t)
        counts[i] = r.n_spikes
        out[i, :len(r.events)] = r.events
    return {"n_spikes": counts, "events": out}


_RUN = {"layer": _run_layer, "classifier": _run_classifier, "recurrent": _run_recurrent, "fit": _run_fit,
        "project": _run_project, "ou": _run_ou, "serve": _run_serve}


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; the operations of the recurrences (about
    8 a neuron-step forward, 16 backward) and of the projections (over the active inputs
    where only these contribute, dense for dx)."""
    c, kind = case, case["kind"]
    if kind == "ou":
        return {"bytes": 4.0 * c["T"] * c["n"], "flops": 40.0 * c["T"] * c["n"]}
    if kind == "serve":
        steps = sum(N * T for N, T, _ in _serve_sizes(c))
        return {"bytes": 16.0 * c["requests"] * c["n_max"], "flops": 48.0 * steps}
    rows, n, n_in = c["batch"] * c["T"], c["n"], c.get("n_in", 0)
    if kind == "project":
        xb = {"u8": 1, "bf16": 2, "f32": 4}[c["x"]]
        return {"bytes": rows * (2.0 * xb * n_in + 4 * n + 4 * n + 4 * n + 4 * n_in) + 12.0 * n * n_in,
                "flops": 2.0 * rows * n * n_in * (1 + 2 * c["density"])}
    if kind == "fit":
        return {"bytes": rows * n * (4.0 + 1 + 4 + c["repeats"] + 4), "flops": rows * n * (24.0 + 8 * c["repeats"])}
    if kind == "recurrent":
        return {"bytes": rows * n * (4.0 + 1 + 4 + 4), "flops": rows * n * 24.0}
    by, fl = rows * (n_in if n_in else 4.0 * n) + 4.0 * n * n_in, rows * n * 8.0 + 2 * rows * n * n_in * c["density"]
    if kind == "classifier":
        C = c["classes"]
        return {"bytes": by + 4.0 * n * n_in + 8.0 * C * n,
                "flops": 2 * fl + rows * n * 8.0 + 4.0 * rows * n * C}
    by += rows * n * (1.0 + (8 if c["traces"] else 0))
    if c["train"]:
        by += rows * n * 4.0 + 4.0 * n * n_in + (rows * n_in * 4.0 if c["dx"] else 0)
        fl += rows * n * 16.0 + 2 * rows * n * n_in * (c["density"] + (1 if c["dx"] else 0))
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def exact(case, seed):
    if case["kind"] == "serve":
        return None            # spike events, whole numbers
    return _EXACT[case["kind"]](case, seed)


def _simulate(I, p, dt, tr, Wrec=None):
    """The standard model step by step. I float64 [B][T][N], bias included (and, with
    Wrec, completed in place by the recurrent current of spikes tr steps earlier)."""
    B, T, N = I.shape
    d64 = {k: (torch.zeros(N, device=DEV) if t is None else t.detach()).double() for k, t in p.items()}
    beta, pa = torch.exp(-dt / d64["tau_mem"]), torch.exp(-dt / d64["tau_adapt"])
    z = lambda dtype=torch.float64: torch.empty(B, T, N, dtype=dtype, device=DEV)
    V, TH, A, S, G = z(), z(), z(), z(torch.bool), z(torch.bool)
    v, a = I.new_zeros(B, N), I.new_zeros(B, N)
    s = torch.zeros(B, N, dtype=torch.bool, device=DEV)
    cnt = torch.full((B, N), tr, dtype=torch.int32, device=DEV)     # steps since the last spike
    for t in range(T):
        if Wrec is not None and t >= tr:
            I[:, t] += S[:, t - tr].double() @ Wrec.t()
        g = cnt >= tr
        v = (beta * v + (1 - beta) * I[:, t] * g) * ~s
        a = pa * a + s
        th = d64["theta0"] + d64["d"] * a
        s = v > th
        cnt = torch.where(s, 1, cnt + 1)
        V[:, t], TH[:, t], A[:, t], S[:, t], G[:, t] = v, th, a, s, g
    return dict(V=V, TH=TH, A=A, S=S, G=G, I=I, beta=beta, pa=pa, d=d64["d"], dt=dt,
                tau_mem=d64["tau_mem"], tau_adapt=d64["tau_adapt"])


def _adjoint(f, gs, want_gI=False, slope=10.0):
    """Detached surrogate adjoint of ``_simulate`` for dL/dS = gs."""
    B, T, N = f["V"].shape
    beta, pa, d, z = f["beta"], f["pa"], f["d"], f["V"].new_zeros(B, N)
    lv, la = z, z
    gb, gp, gd, gt, gbias = z.clone(), z.clone(), z.clone(), z.clone(), z.clone()
    gI = torch.empty_like(f["V"]) if want_gI else None
    for t in range(T - 1, -1, -1):
        V, s = f["V"][:, t], f["S"][:, t]
        q = gs[:, t].double() / (slope * (V - f["TH"][:, t]).abs() + 1) ** 2
        lv = q + beta * ~s * lv
        la = pa * la - d * q
        g = f["G"][:, t]
        gIt = (1 - beta) * g * lv
        if t > 0:
            sp, Vp, Ap = f["S"][:, t - 1], f["V"][:, t - 1], f["A"][:, t - 1]
            g = g & ~sp
            gIt = gIt * ~sp
            gb += ~sp * (Vp - g * f["I"][:, t]) * lv
            gp += Ap * la
        else:
            gb -= g * f["I"][:, t] * lv
        gd -= f["A"][:, t] * q
        gt -= q
        gbias += gIt
        if want_gI:
            gI[:, t] = gIt
    dt = f["dt"]
    return gI, {"grad_tau_mem": gb.sum(0) * beta * dt / f["tau_mem"] ** 2,
                "grad_tau_adapt": gp.sum(0) * pa * dt / f["tau_adapt"] ** 2, "grad_d": gd.sum(0),
                "grad_theta0": gt.sum(0), "grad_bias": gbias.sum(0)}


def _bias(p):
    return 0.0 if p["bias"] is None else p["bias"].detach().double()


def _exact_layer(case, seed):
    s = _layer_inputs(case, seed)
    B, T, n, n_in = case["batch"], case["T"], case["n"], case["n_in"]
    if n_in:
        x64 = s["inp"].view(B * T, n_in).double()
        I = (x64 @ s["W"].double().t()).view(B, T, n)
    else:
        I = s["inp"].double()
    f = _simulate(I + _bias(s["p"]), s["p"], case["dt"], case["tr"])
    out = {"spikes": f["S"].to(torch.uint8)}
    if case["traces"]:
        out.update(v=f["V"], theta=f["TH"])
    if case["train"]:
        gI, g = _adjoint(f, s["gs"], want_gI=n_in > 0)
        out.update(g)
        if n_in:
            out["grad_W"] = gI.view(B * T, n).t() @ x64
        if case["dx"]:
            out["grad_input"] = (gI.view(B * T, n) @ s["W"].double()).view(B, T, n_in)
    return out


def _exact_classifier(case, seed):
    s = _classifier_inputs(case, seed)
    B, T, n, dt = case["batch"], case["T"], case["n"], case["dt"]
    x64 = s["x"].view(B * T, -1).double()
    f = _simulate((x64 @ s["W"].double().t()).view(B, T, n) + _bias(s["p"]), s["p"], dt, case["tr"])
    # the readout's summed membrane in closed form: o = sum_s (1 - beta^(T - s)) (W_r S[s])
    S64 = f["S"].double().view(B * T, n).requires_grad_()
    Wr, tau = s["Wr"].double().requires_grad_(), s["tr"].double().requires_grad_()
    left = torch.arange(T, 0, -1, device=DEV, dtype=torch.float64)[:, None]
    w = 1 - torch.exp(-dt / tau * left)
    o = ((S64 @ Wr.t()).view(B, T, -1) * w).sum(1)
    loss = torch.nn.functional.cross_entropy(o, s["labels"])
    gS, gWr, gtau = torch.autograd.grad(loss, [S64, Wr, tau])
    gI, g = _adjoint(f, gS.view(B, T, n), want_gI=True)
    return {"logits": o.detach(), "loss": loss.detach(),
            "grads": [gI.view(B * T, n).t() @ x64, gWr, gtau, *[g[k] for k in _GRADS]]}


def _exact_recurrent(case, seed):
    s = _recurrent_inputs(case, seed)
    B, T, n, tr = case["batch"], case["T"], case["n"], case["tr"]
    f = _simulate(s["inp"].double(), s["p"], case["dt"], tr, s["Wrec"].double())
    gI, g = _adjoint(f, s["gs"], want_gI=True)
    gw = gI.new_zeros(n, n)
    for b in range(B):
        gw += gI[b, tr:].t() @ f["S"][b, :max(0, T - tr)].double()
    return {"spikes": f["S"].to(torch.uint8), "current": f["I"], "grad_W_rec": gw, **g}


def _exact_fit(case, seed):
    s = _fit_inputs(case, seed)
    B, R, T, n, dt = case["batch"], case["repeats"], case["T"], case["n"], case["dt"]
    f = _simulate(s["inp"].double() + _bias(s["p"]), s["p"], dt, case["tr"])
    a = math.exp(-dt / TAU_VR)
    S = f["S"].to(torch.uint8)

    def filtered():
        e = torch.zeros(B, R, n, dtype=torch.float64, device=DEV)
        for t in range(T):
            e = a * e + (S[:, None, t].double() - s["targets"][:, :, t].double())
            yield t, e

    D2 = torch.zeros(B, R, n, dtype=torch.float64, device=DEV)
    for _, e in filtered():
        D2 += e * e
    D = torch.sqrt(dt / TAU_VR * D2)
    w = torch.where(D > 0, dt / TAU_VR / D.clamp_min(1e-300), 0.0) / (B * R)
    grad = torch.empty(B, T, n, dtype=torch.float64, device=DEV)
    for t, e in filtered():
        grad[:, t] = (w * e).sum(1)
    for t in range(T - 2, -1, -1):
        grad[:, t] += a * grad[:, t + 1]
    _, g = _adjoint(f, grad)
    out = {"spikes": S, "dist": D, "grad_spikes": grad, **g, "params": {}, "m": {}, "v": {}}
    for k, lr, lo, hi in FIT:
        gr = g["grad_" + k]
        out["m"][k], out["v"][k] = 0.1 * gr, 0.001 * gr * gr
        out["params"][k] = (s["p"][k].double() - lr * gr / (gr.abs() + 1e-8)).clamp(lo, hi)
    return out


def _exact_project(case, seed):
    s = _project_inputs(case, seed)
    B, T, n, n_in = case["batch"], case["T"], case["n"], case["n_in"]
    x64, W64, g64 = s["x"].view(-1, n_in).double(), s["W"].double(), s["gI"].view(-1, n).double()
    return {"current": (x64 @ W64.t() + s["bias"].double()).view(B, T, n), "grad_W": g64.t() @ x64,
            "grad_input": (g64 @ W64).view(B, T, n_in)}


def _philox(c0, c1, key):
    """Philox4x32-10 of counter (c0, c1, 0, 0) on int64 tensors holding 32-bit words."""
    M = 0xFFFFFFFF
    c = [c0, c1, torch.zeros_like(c0), torch.zeros_like(c0)]
    k0, k1 = key & M, (key >> 32) & M

    def mul(m, x):            # (high, low) words of the 64-bit product, in 16-bit pieces
        lo, hi = (x & 0xFFFF) * m, (x >> 16) * m
        s = hi + (lo >> 16)
        return s >> 16 & M, ((s & 0xFFFF) << 16) | (lo & 0xFFFF)

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c


def _exact_ou(case, seed):
    T, n, dt = case["T"], case["n"], case["dt"]
    q = torch.arange((T + 3) // 4, device=DEV)[:, None].expand(-1, n).contiguous()
    w = _philox(q, torch.arange(n, device=DEV).expand_as(q).contiguous(), seed)
    z = torch.empty(q.shape[0], 4, n, dtype=torch.float64, device=DEV)
    for j in (0, 1):
        r = torch.sqrt(-2.0 * torch.log((w[2 * j].double() + 1.0) * 2.0**-32))
        ang = 2.0 * math.pi * (w[2 * j + 1].double() * 2.0**-32)
        z[:, 2 * j], z[:, 2 * j + 1] = r * torch.cos(ang), r * torch.sin(ang)
    x = z.view(-1, n)[:T]
    e = math.exp(-dt / 5.0)
    x[1:] *= math.sqrt(1.0 - e * e)
    x *= 0.5
    for t in range(1, T):
        x[t] += e * x[t - 1]
    return x + float(np.float32(0.8))     # the call takes the mean as a float


_EXACT = {"layer": _exact_layer, "classifier": _exact_classifier, "recurrent": _exact_recurrent, "fit": _exact_fit,
          "project": _exact_project, "ou": _exact_ou}
