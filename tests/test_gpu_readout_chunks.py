"""The readout's recurrence on as many chunks as its classes allow (64 at up to 16 classes,
fewer above, several workgroups past 32): T below, at and above the chunks and their
registers, against the oracle to the bars of the layer tests."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log, np_
from parity import check_grad
from paper_2311_11390_amd.synth import bernoulli_spikes, normal_weights, rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [1, 2, 10, 16, 17, 20, 32, 33])
@pytest.mark.parametrize("T", [1, 63, 65, 769, 2000])
def test_readout_chunks(C, T):
    import torch

    from paper_2311_11390_amd import alif
    B, H, dt = 2, 52, 1.0
    log(f"[readout] C={C} T={T}")
    g = rng(1000 * C + T)
    S, Wr = bernoulli_spikes(g, (B, T, H), 0.1), normal_weights(g, C, H)
    tau = g.uniform(10.0, 30.0, C).astype(np.float32)
    go = g.standard_normal((B, C)).astype(np.float32)
    St, Wt, tt = (torch.as_tensor(a, device="cuda") for a in (S, Wr, tau))
    o, ws = alif.readout_forward(St, Wt, tt, dt)
    gS, gW, gt = alif.readout_backward(St, Wt, tt, dt, torch.as_tensor(go, device="cuda"), ws)
    torch.cuda.synchronize()
    Ir = S.astype(np.float64) @ Wr.astype(np.float64).T
    np.testing.assert_allclose(np_(o), oracle.readout_forward(Ir, tau, dt)["o"], rtol=1e-5, atol=1e-4)
    rb = oracle.readout_backward(Ir, tau, dt, go)
    check_grad("readout grad_spikes", np_(gS), rb["gIr"] @ Wr.astype(np.float64))
    check_grad("readout grad_W", np_(gW), np.einsum("btc,bth->ch", rb["gIr"], S.astype(np.float64)))
    if T > 1:
        check_grad("readout grad_tau", np_(gt), rb["g_tau_r"])
