"""FP32 projections whose floats reach past 2^60, where tiles are done over by FP32 MFMA:
finite results against FP64 products within (K + 8) 2^-24 of the sum of magnitudes (an FP32
accumulation of K products in any order), with remainders of the tile, of the steps of k and
of K splits; and beside tiles that are not done over."""
import numpy as np
import pytest

from gpu_helpers import log, np_
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("xd", ["uint8", "bfloat16", "float32"])
@pytest.mark.parametrize("B,T,K,N", [(1, 1, 4, 4), (1, 129, 36, 132), (2, 700, 132, 260), (1, 3001, 20, 64)])
@pytest.mark.parametrize("where", ["all", "one"])
def test_past_two_to_the_sixty(B, T, K, N, xd, where):
    import torch

    from paper_2311_11390_amd import alif
    log(f"[split range] {B}x{T} {K}->{N} {xd} {where}")
    g = rng(T + K + N)
    x = g.integers(0, 2, (B, T, K)).astype(np.float32)
    W, gI = (g.standard_normal(s).astype(np.float32) for s in ((N, K), (B, T, N)))
    if where == "all":
        W, gI = W * np.float32(2.0**61), gI * np.float32(2.0**40)     # (products stay below 2^124)
        W[0, 0], gI[0, 0, 0] = 2.0**62, 2.0**60
    else:
        W[N - 1, K - 1], gI[B - 1, T - 1, N - 1] = 2.0**61, -(2.0**60)
    xt = torch.as_tensor(x).to(getattr(torch, xd)).cuda()
    Wt, gt = torch.as_tensor(W, device="cuda"), torch.as_tensor(gI, device="cuda")
    got = (alif.input_current(xt, Wt), alif.weight_grad(gt, xt), alif.input_grad(gt, Wt, alif._INPUT_KIND[xt.dtype]))
    torch.cuda.synchronize()
    x2, W2, g2 = x.reshape(-1, K).astype(np.float64), W.astype(np.float64), gI.reshape(-1, N).astype(np.float64)
    for name, o, (a, b) in zip(("current", "dW", "dx"), got, ((x2, W2.T), (g2.T, x2), (g2, W2))):
        ref, s = a @ b, np.abs(a) @ np.abs(b)
        err = np.abs(np_(o).astype(np.float64).reshape(ref.shape) - ref)
        bound = (a.shape[1] + 8) * 2.0**-24 * s
        assert (err <= bound).all(), f"{name}: {(err / np.maximum(bound, 1e-300)).max():.2f} of the bound"
