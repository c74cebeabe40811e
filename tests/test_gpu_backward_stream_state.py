"""The streaming backward from any initial state and beside infinite gradients: the
parameter gradients without dL/dI against the block backward's (asked for dL/dI at sizes
where its rule keeps the block kernel; the path is asserted)."""
import numpy as np
import pytest

from dispatch import stream_chunks, streams_dI
from gpu_helpers import driven_current, gpu_forward, log, np_, random_params
from parity import check_grad
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu

_ALL = ("grad_tau_mem", "grad_tau_adapt", "grad_d", "grad_theta0", "grad_bias")


def _both(B, T, N, TR, seed, init, gS):
    import torch

    from paper_2311_11390_amd import alif
    assert not streams_dI(B, T, N, TR)
    I = driven_current(seed, B, T, N)
    prm = random_params(seed, N, tm=(2.0, 30.0), bias=(-0.3, 0.3))
    f, It, P = gpu_forward(I, prm, 2.0 / TR, 2.0, traces=False, save=True, init=init)
    g = torch.as_tensor(gS, device="cuda")
    a = alif.backward(f, It, P, grad_spikes=g)
    b = alif.backward(f, It, P, grad_spikes=g, want_grad_current=True)
    torch.cuda.synchronize()
    return {k: np_(a[k]).astype(np.float64) for k in _ALL}, {k: np_(b[k]).astype(np.float64) for k in _ALL}


@pytest.mark.parametrize("TR", [2, 3, 4, 5, 8, 16, 32, 64])
def test_any_initial_state(TR):
    """Initial states whose membrane is not zero after a spike (in the last step of the block
    before too): the forward lets it decay from there, and so do its gradients."""
    import torch
    B, N, T = 3, 130, 3 * TR
    log(f"[stream state] T_R={TR}")
    g = rng(990 + TR)
    t = lambda x: torch.as_tensor(x, device="cuda")
    ts = g.integers(0, TR + 1, (B, N)).astype(np.int32)
    ts[:, ::3] = TR
    init = {"v": t(g.uniform(0.1, 0.8, (B, N))), "a": t(g.uniform(0.0, 2.0, (B, N))), "ts": t(ts)}
    a, b = _both(B, T, N, TR, 990 + TR, init, g.standard_normal((B, T, N)).astype(np.float32))
    for k in _ALL:
        check_grad(k, a[k], b[k])


@pytest.mark.parametrize("TR", [3, 8, 64])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_bias_gradient_beside_infinite_gradients_of_masked_steps(TR, bad):
    """A refractory step passes no input on, so its dL/dS does not reach the bias."""
    import torch
    B, N, T = 2, 66, 3 * TR
    log(f"[stream masked] T_R={TR} {bad}")
    g = rng(995 + TR)
    t = lambda x: torch.as_tensor(x, device="cuda")
    init = {"v": t(np.zeros((B, N))), "a": t(g.uniform(0.0, 2.0, (B, N))), "ts": t(np.full((B, N), TR, np.int32))}
    gS = g.standard_normal((B, T, N)).astype(np.float32)
    gS[:, 0, ::2] = bad      # the step after the last block's spike
    a, b = _both(B, T, N, TR, 995 + TR, init, gS)
    assert np.isfinite(b["grad_bias"]).all()
    check_grad("grad_bias", a["grad_bias"], b["grad_bias"])
    for k in _ALL:
        np.testing.assert_array_equal(np.isfinite(a[k]), np.isfinite(b[k]), err_msg=k)
        ok = np.isfinite(b[k])
        check_grad(k, a[k][ok], b[k][ok])


@pytest.mark.parametrize("TR,T", [(2, 201), (5, 203), (20, 410), (40, 803)])
def test_resumed_run_in_several_chunks(TR, T):
    """A run resumed from a saved state (live masks, adaptation), cut into chunks, against the
    block backward on the same piece."""
    import torch
    B, N = 128, 512
    assert stream_chunks(B, T, N, TR) > 1
    log(f"[stream state] resumed T_R={TR} T={T}")
    I = driven_current(940 + TR, B, 10 * TR, N)
    prm = random_params(940 + TR, N, tm=(2.0, 30.0), bias=(-0.3, 0.3))
    f, _, _ = gpu_forward(I, prm, 2.0 / TR, 2.0, traces=False, want_final=True)
    assert (f["final"]["ts"] > 1).any() and (f["final"]["a"] > 0).any()
    gS = rng(941 + TR).standard_normal((B, T, N)).astype(np.float32)
    a, b = _both(B, T, N, TR, 940 + TR, f["final"], gS)
    for k in _ALL:
        check_grad(k, a[k], b[k])
