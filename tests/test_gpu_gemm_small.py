"""A layer's FP32 currents from few rows or unaligned rows (a wave takes 16 x 16, 16 x 32 or
32 x 32 of the product straight from memory) against the tiled path's, which the same rows
take as part of a larger input: both sum by the same matrix instruction over increasing k,
so they agree bit for bit. Row and column remainders of every tile, k of every remainder
by 4 and around the steps in flight, the three input types; unaligned rows against the
oracle's projection to the FP32 sum's bound."""
import numpy as np
import pytest

from gpu_helpers import log, random_params, to_dev

pytestmark = pytest.mark.gpu


def _current(x, W, P):
    from paper_2311_11390_amd import alif
    return alif.forward(x, P, 0.5, 2.0, W, save=True)["current"]


@pytest.mark.parametrize("dtype", ["uint8", "bfloat16", "float32"])
@pytest.mark.parametrize("N,K", [(1, 4), (20, 60), (100, 200), (33, 64), (129, 132), (512, 256), (65, 700)])
def test_small_equals_tiled(dtype, N, K):
    import torch
    log(f"[small gemm] {dtype} N={N} K={K}")
    M = 600_000 // N + 17
    g = torch.Generator(device="cuda").manual_seed(N + K)
    x = (torch.rand(1, M, K, generator=g, device="cuda") < 0.2).to(getattr(torch, dtype))
    W = torch.randn(N, K, generator=g, device="cuda")
    P = to_dev(random_params(K, N, bias=(-0.3, 0.3)))
    big = _current(x, W, P)
    for m in (1, 15, 16, 17, 33, 260_000 // N, 500_000 // N):
        assert torch.equal(_current(x[:, :m].contiguous(), W, P)[0], big[0, :m]), m


@pytest.mark.parametrize("dtype", ["uint8", "bfloat16", "float32"])
@pytest.mark.parametrize("M,N,K", [(3, 5, 1), (17, 33, 3), (300, 20, 61), (1000, 300, 203), (2001, 513, 130)])
def test_unaligned_rows(dtype, M, N, K):
    import torch
    log(f"[small gemm] unaligned {dtype} {M}x{N}x{K}")
    g = torch.Generator(device="cuda").manual_seed(M)
    x = (torch.rand(1, M, K, generator=g, device="cuda") < 0.2).to(getattr(torch, dtype))
    W = torch.randn(N, K, generator=g, device="cuda")
    prm = random_params(K, N, bias=(-0.3, 0.3))
    got = _current(x, W, to_dev(prm))[0].cpu().numpy().astype(np.float64)
    xs, Ws = x[0].float().cpu().numpy().astype(np.float64), W.cpu().numpy().astype(np.float64)
    b = np.asarray(prm.bias, np.float64)
    want = xs @ Ws.T + b
    bound = (K + 2) * 2.0 ** -24 * (np.abs(xs) @ np.abs(Ws).T + np.abs(b))
    assert (np.abs(got - want) <= bound).all()
