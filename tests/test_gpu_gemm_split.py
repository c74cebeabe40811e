"""FP32 projections on the bfloat16 matrix cores (three-piece operands) through
alif_input_current, alif_weight_grad and alif_input_grad, against FP64 products.

Bound, element by element, with S = sum over k of |a| |b|: an FP32 accumulation of K
products of up to three pieces each, in any order, is within (K + 3) 2^-24 S; the product
terms left out of float x float are below 2^-22 of a product (2^-7 2^-16 twice, and less),
4 more units: (K + 8) 2^-24 S covers both, the bias and the final sum."""
import numpy as np
import pytest

from gpu_helpers import log, np_
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu

_DT = {"u8": "uint8", "bf16": "bfloat16", "f32": "float32"}


def _inputs(seed, B, T, K, N, xd):
    import torch
    g = rng(seed)
    x = torch.as_tensor(g.integers(0, 3, (B, T, K)).astype(np.float32) if xd == "u8"
                        else g.standard_normal((B, T, K)).astype(np.float32)).to(getattr(torch, _DT[xd])).cuda()
    W, gI, bias = (torch.as_tensor(g.standard_normal(s).astype(np.float32) * c).cuda()
                   for s, c in (((N, K), 1.0), ((B, T, N), 1e-3), ((N,), 1.0)))
    return x, W, gI, bias


def _run(x, W, gI, bias):
    import torch

    from paper_2311_11390_amd import alif
    out = (alif.input_current(x, W, bias), alif.weight_grad(gI, x), alif.input_grad(gI, W, alif._INPUT_KIND[x.dtype]))
    torch.cuda.synchronize()
    return [np_(t).astype(np.float64) for t in out]


def _pairs(x, W, gI, bias):
    """(a, b, bias) with result a @ b of each call, float64."""
    K, N = x.shape[2], W.shape[0]
    x2, W2, g2 = np_(x).astype(np.float64).reshape(-1, K), np_(W).astype(np.float64), np_(gI).astype(np.float64).reshape(-1, N)
    return (x2, W2.T, np_(bias).astype(np.float64)), (g2.T, x2, 0.0), (g2, W2, 0.0)


# tile edges of rows and columns (128), of the stage (16 and 32 k), of a single row, the
# smallest vector-aligned widths, and long K splits
@pytest.mark.parametrize("xd", ["u8", "bf16", "f32"])
@pytest.mark.parametrize("B,T,K,N", [(1, 1, 4, 4), (1, 127, 16, 20), (1, 129, 36, 128), (2, 64, 128, 132),
                                     (1, 300, 132, 260), (3, 700, 200, 64), (1, 33, 64, 512)])
def test_split_projections(B, T, K, N, xd):
    log(f"[split] {B}x{T} {K}->{N} {xd}")
    ops = _inputs(K + N + T, B, T, K, N, xd)
    for name, got, (a, b, c) in zip(("current", "dW", "dx"), _run(*ops), _pairs(*ops)):
        ref = a @ b + c
        bound = (a.shape[1] + 8) * 2.0**-24 * (np.abs(a) @ np.abs(b) + np.abs(c)) + 1e-36
        err = np.abs(got.reshape(ref.shape) - ref)
        assert (err <= bound).all(), f"{name}: {np.max(err / bound):.2f} of the bound"


@pytest.mark.parametrize("xd", ["u8", "f32"])
def test_split_projections_infinite_and_huge(xd):
    """Infinities, NaNs and magnitudes near the top of the range come out as they do
    from FP32 multiply-adds: the same NaNs and infinities, the rest within the bound."""
    B, T, K, N = 1, 200, 96, 136
    log(f"[split] infinities {xd}")
    x, W, gI, bias = _inputs(7, B, T, K, N, xd)
    x[0, 150, 4] = 1
    W[3, 4], W[3, 5], W[130, 7], W[131, 9], W[5, 1] = float("inf"), float("-inf"), 3.0e38, 1e30, float("nan")
    gI[0, 2, 3], gI[0, 140, 130], gI[0, 141, 8] = float("inf"), -3.1e38, float("nan")
    with np.errstate(all="ignore"):
        for name, got, (a, b, c) in zip(("current", "dW", "dx"), _run(x, W, gI, bias), _pairs(x, W, gI, bias)):
            ref = a @ b + c
            ref = np.where(np.abs(ref) > 3.4028235677973366e38, np.sign(ref) * np.inf, ref)
            got = got.reshape(ref.shape)
            bound = (a.shape[1] + 8) * 2.0**-24 * (np.abs(a) @ np.abs(b) + np.abs(c))
            np.testing.assert_array_equal(np.isnan(got), np.isnan(ref), err_msg=name)
            np.testing.assert_array_equal(np.isinf(got), np.isinf(ref), err_msg=name)
            fin = np.isfinite(ref)
            assert np.isinf(ref).any() and fin.any()
            assert (np.sign(got) == np.sign(ref))[np.isinf(ref)].all()
            assert (np.abs(got - ref)[fin] <= bound[fin]).all(), name
