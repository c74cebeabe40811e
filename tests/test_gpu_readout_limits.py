"""The readout's backward at the limits of its inputs: a time constant of zero (no
memory), of infinity (no leak) or negative (growth), and an infinite or NaN logit gradient,
against the sequential recurrence lam[t] = g + beta lam[t+1], gI_r = (1 - beta) lam in FP64.
One class that reads its hidden neurons with weight one, so grad_spikes is gI_r. One chunk
of time and several, steps beside empty chunks."""
import numpy as np
import pytest

from gpu_helpers import log, np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 40, 700])
@pytest.mark.parametrize("tau", [20.0, 0.0, 1e-3, float("inf"), -400.0])
def test_backward_at_the_limits(T, tau):
    import torch

    from paper_2311_11390_amd import alif
    H, dt = 4, 1.0
    log(f"[readout limits] T={T} tau={tau}")
    go = np.array([0.5, -0.25, np.inf, -np.inf, np.nan])
    B = len(go)
    S = torch.zeros(B, T, H, dtype=torch.uint8, device="cuda")
    W, tr = torch.ones(1, H, device="cuda"), torch.full((1,), tau, device="cuda")
    _, ws = alif.readout_forward(S, W, tr, dt)
    gS, _, _ = alif.readout_backward(S, W, tr, dt, torch.as_tensor(go.astype(np.float32)[:, None], device="cuda"), ws)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        lb = -dt / np.float64(tau)
        beta, omb = np.exp(lb), -np.expm1(lb)
        lam, ref = np.zeros(B), np.zeros((B, T))
        for t in range(T - 1, -1, -1):
            lam = go + beta * lam
            ref[:, t] = omb * lam
    got = np_(gS).astype(np.float64)
    for h in range(H):
        for b in range(B):
            # FP64 sums rounded once to float (a chunk's carry is a closed form of the same sum)
            np.testing.assert_allclose(got[b, :, h], ref[b], rtol=1e-6, atol=0, err_msg=f"g {go[b]}")
