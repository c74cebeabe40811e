"""The readout's products for few classes (straight from the spikes, without GEMM tiles) and
their limits: every class count around the paddings, hidden neurons below, at and above a
workgroup's columns and of no multiple of four (GEMMs), rows around the staged tiles and the
shares of the weight gradient, the three spike types, misaligned spikes; against the oracle
to the bars of the layer tests."""
import numpy as np
import pytest

import oracle
from gpu_helpers import log, np_
from parity import check_grad
from paper_2311_11390_amd.synth import bernoulli_spikes, normal_weights, rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,H,C,dtype,shift", [
    (1, 1, 4, 1, "uint8", 0), (2, 33, 252, 8, "float32", 0), (1, 64, 256, 9, "bfloat16", 0), (3, 43, 260, 16, "uint8", 0),
    (1, 65, 512, 17, "float32", 0), (2, 100, 20, 24, "bfloat16", 0), (1, 130, 1024, 25, "uint8", 0),
    (2, 8200, 64, 20, "float32", 0), (5, 4001, 36, 10, "uint8", 0), (2, 50, 100, 33, "float32", 0),
    (1, 77, 300, 48, "bfloat16", 0), (1, 60, 64, 49, "float32", 0), (2, 40, 63, 20, "uint8", 0),
    (2, 40, 64, 20, "uint8", 1), (2, 40, 64, 20, "bfloat16", 1), (2, 40, 64, 20, "float32", 1)])
def test_readout_products(B, T, H, C, dtype, shift):
    import torch

    from paper_2311_11390_amd import alif
    log(f"[readout products] B={B} T={T} H={H} C={C} {dtype} shift={shift}")
    g = rng(B + 10 * T + H + 1000 * C)
    S, Wr = bernoulli_spikes(g, (B, T, H), 0.1), normal_weights(g, C, H)
    tau = g.uniform(10.0, 30.0, C).astype(np.float32)
    go = g.standard_normal((B, C)).astype(np.float32)
    buf = torch.zeros(S.size + shift, dtype=getattr(torch, dtype), device="cuda")
    St = buf[shift:].view(B, T, H)
    St.copy_(torch.as_tensor(S))
    Wt, tt = torch.as_tensor(Wr, device="cuda"), torch.as_tensor(tau, device="cuda")
    o, ws = alif.readout_forward(St, Wt, tt, 1.0)
    gS, gW, gt = alif.readout_backward(St, Wt, tt, 1.0, torch.as_tensor(go, device="cuda"), ws)
    torch.cuda.synchronize()
    Ir = S.astype(np.float64) @ Wr.astype(np.float64).T
    ref = oracle.readout_forward(Ir, tau, 1.0)["o"]
    np.testing.assert_allclose(np_(o), ref, rtol=1e-5, atol=1e-4)
    rb = oracle.readout_backward(Ir, tau, 1.0, go)
    check_grad("readout grad_spikes", np_(gS), rb["gIr"] @ Wr.astype(np.float64))
    check_grad("readout grad_W", np_(gW), np.einsum("btc,bth->ch", rb["gIr"], S.astype(np.float64)))
