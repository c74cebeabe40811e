"""Both kernels of the detached backward with dL/dI against the oracle's sequential adjoint,
each at sizes its rule really sends to it: the block kernel at every segmentation (its
largest call at these widths that does not stream), the streaming one from its smallest
call on, in several chunks and in one (a card full of rows). dL/dI and the parameter
gradients to the gradient bar of parity.check_grad."""
import numpy as np
import pytest

import oracle
from dispatch import stream_chunks, streams_dI
from gpu_helpers import driven_current, gpu_forward, log, np_, random_params
from parity import check_forward, check_grad
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu

_NAMES = [("grad_tau_mem", "g_tau_m"), ("grad_tau_adapt", "g_tau_a"), ("grad_d", "g_d"), ("grad_theta0", "g_theta0")]


def _check(B, T, N, TR, form, what):
    import torch

    from paper_2311_11390_amd import alif
    dt = 2.0 / TR
    log(f"[bwd path] {what} T_R={TR} B={B} T={T} N={N} gradients {form}")
    I = driven_current(1200 + TR, B, T, N)
    prm = random_params(1200 + TR, N, tm=(2.0, 30.0), bias=(-0.3, 0.3))
    g = rng(1201 + TR)
    gs = {k: g.standard_normal((B, T, N)).astype(np.float32) if k in form else None for k in "svt"}
    tt = {k: None if a is None else torch.as_tensor(a, device="cuda") for k, a in gs.items()}
    f, It, P = gpu_forward(I, prm, dt, 2.0, traces=False, save=True)
    out = alif.backward(f, It, P, grad_spikes=tt["s"], grad_v=tt["v"], grad_theta=tt["t"], want_grad_current=True)
    torch.cuda.synchronize()
    orc = check_forward(np_(f["spikes"]), I, prm, dt, 2.0)["oracle"]
    ob = oracle.alif_backward(orc, dt, 10.0, gS=gs["s"], gV=gs["v"], gTH=gs["t"])
    check_grad("grad_current", np_(out["grad_current"]), ob["gI"])
    for k, ko in _NAMES:
        check_grad(k, np_(out[k]), ob[ko])
    check_grad("grad_bias", np_(out["grad_bias"]), ob["gI"].sum(axis=(0, 1)))


def _blocks(B, N, TR, gvt, stream):
    """Steps of the largest call of up to 12 blocks that does not stream, or of the smallest that does."""
    T = lambda nb: nb * TR + TR // 2 + 1
    if stream:
        return T(next(nb for nb in range(1, 3000) if streams_dI(B, T(nb), N, TR, gvt)))
    return T(max(nb for nb in range(1, 13) if not streams_dI(B, T(nb), N, TR, gvt)))


_TRS = [2, 3, 4, 5, 6, 7, 8, 11, 12, 16, 20, 23, 24, 31, 32, 40, 47, 48, 50, 64, 80, 96, 100, 104, 110, 112, 120, 127, 128]


@pytest.mark.parametrize("TR", _TRS)
@pytest.mark.parametrize("form", ["s", "svt"])
def test_block_kernel(TR, form):
    B, N = 5, 131
    T = _blocks(B, N, TR, form != "s", False)
    assert not streams_dI(B, T, N, TR, form != "s")
    _check(B, T, N, TR, form, "block")


@pytest.mark.parametrize("TR", _TRS)
@pytest.mark.parametrize("form", ["s", "svt"])
def test_streaming_kernels(TR, form):
    B, N = 2, 67
    T = _blocks(B, N, TR, form != "s", True)
    assert streams_dI(B, T, N, TR, form != "s") and stream_chunks(B, T, N, TR) > 1
    _check(B, T, N, TR, form, "streaming")


@pytest.mark.parametrize("TR,form", [(50, "s"), (100, "s"), (100, "svt"), (128, "svt")])
def test_streaming_kernels_in_one_chunk(TR, form):
    B, N = 2200, 3
    T = 4 * TR + 3
    assert streams_dI(B, T, N, TR, form != "s") and stream_chunks(B, T, N, TR) == 1
    _check(B, T, N, TR, form, "streaming, one chunk")
