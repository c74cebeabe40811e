"""Gradients of a BF16 layer at sizes where an FP32 layer's backward streams: dL/dI is
the block kernel's, bit for bit, because the projections' gradients round it to
bfloat16 (1e-6 beside it flips elements over a rounding boundary, 1e-4 in dW and dx).
The block kernel's dL/dI comes from the same rows as part of a batch that it takes in
FP32 too: a row's result does not depend on the others."""
import numpy as np
import pytest

from dispatch import streams_dI
from gpu_helpers import log, np_, random_params, to_dev
from paper_2311_11390_amd.synth import bernoulli_spikes, normal_weights, rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("TR", [2, 4, 5, 10])
@pytest.mark.parametrize("N", [96, 67])
def test_bf16_layer_gradients_come_from_the_block_kernel(TR, N):
    import torch

    from paper_2311_11390_amd import _lib as L
    from paper_2311_11390_amd import alif
    B, T, n_in, rep, dt = 2, 400, 72, 256, 2.0 / TR
    assert streams_dI(B, T, N, TR) and not streams_dI(B * rep, T, N, TR)
    g = rng(4000 + TR + N)
    log(f"[bf16 layer gradients] T_R={TR} N={N}")
    prm = random_params(4000 + TR, N, bias=(0.5, 1.5))
    P = to_dev(prm)
    x = torch.as_tensor(bernoulli_spikes(g, (B, T, n_in), 0.1).astype(np.uint8), device="cuda")
    W = torch.as_tensor(normal_weights(g, N, n_in) * 4.0, device="cuda")
    gS = torch.as_tensor(g.standard_normal((B, T, N)).astype(np.float32), device="cuda")
    f = alif.forward(x, P, dt, 2.0, W, gemm_precision=L.GEMM_BF16, save=True)
    a = alif.backward(f, x, P, W, grad_spikes=gS, want_grad_input=True, want_grad_W=True)
    b = alif.backward(f, x, P, W, grad_spikes=gS, want_grad_input=True, want_grad_W=True, want_grad_current=True)
    Pn = alif.Params(P.tau_mem, P.tau_adapt, P.d, P.theta0)
    cur = f["current"].repeat(rep, 1, 1)
    fb = alif.forward(cur, Pn, dt, 2.0, save=True)
    gI = alif.backward(fb, cur, Pn, grad_spikes=gS.repeat(rep, 1, 1), want_grad_current=True)["grad_current"][:B]
    torch.cuda.synchronize()
    gI = gI.contiguous()
    assert torch.equal(b["grad_current"], gI)
    gin = alif.input_grad(gI, W, gemm_precision=L.GEMM_BF16)
    r = gI.bfloat16().double().reshape(-1, N)
    xd = x.double().reshape(-1, n_in)
    dW, terms = r.T @ xd, r.abs().T @ xd
    for out in (a, b):
        assert torch.equal(out["grad_input"], gin)
        # FP32 sums of B T exact products
        err = (out["grad_W"].double() - dW).abs()
        assert bool((err <= (B * T + 8) * 2.0 ** -24 * terms).all()), float(err.max())
        for k in ("grad_tau_mem", "grad_tau_adapt", "grad_d", "grad_theta0", "grad_bias"):
            assert np.isfinite(np_(out[k])).all()
