"""FP32 projections from bfloat16 pieces where a result has one or two terms (rows of the
input gradient in which one or two neurons have a gradient, the weight gradient of one or
two rows): no further from 64 bits than FP32 multiply-adds allow, so none of the piece
products that reach a product's last bit is missing.

One term: the pieces hold all 24 bits and their products are exact; what is left out is
3 2^-34 of the product (l l, 2^-17 2^-17 of the binades, a product being at least 1 of
them), the small pieces' sum (2^-6 of the product) is rounded seven times, and the result
once: (1 + 2^-3) 2^-24 |p|. Two terms: each is summed into the accumulators besides, and a
multiply-add may drop the bits below its larger operand: 2^-23 of |p1| + |p2| + |s|."""
import numpy as np
import pytest

from gpu_helpers import log, np_
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu


def _check(name, terms, got):
    """terms [t][...] float64 products, got their sum on the device"""
    ref, mag = terms.sum(0), np.abs(terms).sum(0)
    bound = 2.0**-24 * 1.125 * mag if terms.shape[0] == 1 else 2.0**-23 * (mag + np.abs(ref))
    err = np.abs(got.astype(np.float64) - ref)
    assert (err <= bound).all(), f"{name}: {(err / bound).max():.2f} of the bound"


@pytest.mark.parametrize("terms", [1, 2])
def test_input_gradient_of_few_neurons(terms):
    import torch

    from paper_2311_11390_amd import alif
    B, T, K, N = 2, 600, 256, 64
    log(f"[split few] dx, {terms} neurons a row")
    g = rng(800 + terms)
    W = g.uniform(0.5, 2.0, (N, K)).astype(np.float32) * g.choice([-1.0, 1.0], (N, K)).astype(np.float32)
    gI = np.zeros((B * T, N), np.float32)
    rows = np.arange(B * T)
    cols = np.stack([(rows * 7 + 31 * t) % N for t in range(terms)])
    vals = g.uniform(0.5, 2.0, (terms, B * T)).astype(np.float32)
    for t in range(terms):
        gI[rows, cols[t]] = vals[t]
    out = alif.input_grad(torch.as_tensor(gI.reshape(B, T, N), device="cuda"), torch.as_tensor(W, device="cuda"))
    torch.cuda.synchronize()
    _check("dx", vals[:, :, None].astype(np.float64) * W[cols].astype(np.float64), np_(out).reshape(-1, K))


@pytest.mark.parametrize("T", [1, 2])
def test_weight_gradient_of_few_rows(T):
    import torch

    from paper_2311_11390_amd import alif
    K, N = 512, 512
    log(f"[split few] dW of {T} rows")
    g = rng(810 + T)
    x, gI = (g.uniform(0.5, 2.0, (1, T, n)).astype(np.float32) for n in (K, N))
    x *= g.choice([-1.0, 1.0], x.shape).astype(np.float32)
    out = alif.weight_grad(torch.as_tensor(gI, device="cuda"), torch.as_tensor(x, device="cuda"))
    torch.cuda.synchronize()
    _check("dW", gI[0].astype(np.float64)[:, :, None] * x[0].astype(np.float64)[:, None, :], np_(out))
