"""The streaming backward with dL/dI (a forward pass that leaves each step's source, a
pass backward in time over the same chunks): dL/dI and the parameter gradients against the
oracle's sequential adjoint on the teacher-forced forward, to the gradient bar of
parity.check_grad. T_R on both sides of every grouping, T with a ragged last block, one
chunk and several, neuron tails, subsets of the incoming gradients (none: zeros), a run
that starts from a saved state inside a refractory period."""
import numpy as np
import pytest

import oracle
from gpu_helpers import driven_current, gpu_forward, log, np_, random_params
from parity import check_forward, check_grad
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu

_NAMES = [("grad_tau_mem", "g_tau_m"), ("grad_tau_adapt", "g_tau_a"), ("grad_d", "g_d"), ("grad_theta0", "g_theta0")]


@pytest.mark.parametrize("TR", [2, 3, 4, 5, 6, 7, 8, 9, 16, 23, 47, 100, 128])
@pytest.mark.parametrize("form", ["s", "svt", "t", ""])
def test_streamed_current_gradient_matches_oracle(TR, form):
    import torch

    from paper_2311_11390_amd import alif
    B, N, dt = 2, 67, 2.0 / TR
    T = (1 if form == "t" else 6) * max(60, 3 * TR) + TR // 2 + 1     # "t": one chunk
    I = driven_current(950 + TR, B, T, N)
    prm = random_params(950 + TR, N, tm=(2.0, 30.0), bias=(-0.3, 0.3))
    g = rng(951 + TR)
    gs = {k: g.standard_normal((B, T, N)).astype(np.float32) if k in form else None for k in "svt"}
    log(f"[stream dI] T_R={TR} T={T} gradients {form!r}")
    f, It, P = gpu_forward(I, prm, dt, 2.0, traces=False, save=True)
    tt = {k: None if a is None else torch.as_tensor(a, device="cuda") for k, a in gs.items()}
    out = alif.backward(f, It, P, grad_spikes=tt["s"], grad_v=tt["v"], grad_theta=tt["t"], want_grad_current=True)
    torch.cuda.synchronize()
    if not form:
        assert all(torch.count_nonzero(v) == 0 for k, v in out.items() if v is not None)
        return
    orc = check_forward(np_(f["spikes"]), I, prm, dt, 2.0)["oracle"]
    ob = oracle.alif_backward(orc, dt, 10.0, gS=gs["s"], gV=gs["v"], gTH=gs["t"])
    check_grad("grad_current", np_(out["grad_current"]), ob["gI"])
    for k, ko in _NAMES:
        check_grad(k, np_(out[k]), ob[ko])
    check_grad("grad_bias", np_(out["grad_bias"]), ob["gI"].sum(axis=(0, 1)))


@pytest.mark.parametrize("TR", [2, 5, 40])
def test_resumed_run_equals_the_whole_run(TR):
    """dL/dI of the second half alone (started inside refractory periods) equals the whole
    run's over that half: dL/dI depends on the steps after it, so only the chunk borders differ."""
    import torch

    from paper_2311_11390_amd import alif
    B, N, dt, T = 2, 130, 2.0 / TR, 40 * TR
    I = driven_current(980 + TR, B, 2 * T, N)
    prm = random_params(980 + TR, N, tm=(2.0, 30.0))
    log(f"[stream dI] resumed T_R={TR}")
    f0, I0, P = gpu_forward(I, prm, dt, 2.0, traces=False, save=True)
    f1, _, _ = gpu_forward(I[:, :T], prm, dt, 2.0, traces=False, want_final=True)
    assert (f1["final"]["ts"] > 1).any() and (f1["final"]["a"] > 0).any()
    f2, It, _ = gpu_forward(I[:, T:], prm, dt, 2.0, traces=False, save=True, init=f1["final"])
    assert torch.equal(f2["spikes"], f0["spikes"][:, T:])
    gs = torch.as_tensor(rng(981).standard_normal((B, 2 * T, N)).astype(np.float32), device="cuda")
    whole = alif.backward(f0, I0, P, grad_spikes=gs, want_grad_current=True)
    half = alif.backward(f2, It, P, grad_spikes=gs[:, T:].contiguous(), want_grad_current=True)
    torch.cuda.synchronize()
    check_grad("grad_current", np_(half["grad_current"]), np_(whole["grad_current"])[:, T:].astype(np.float64))
