"""alif_backward_noalloc where the streaming backward's chunks fill most of the static
scratch: as many chunks as with a caller's workspace, so the same bits, for every
gradient, with and without dL/dI, at T_R whose last segment is partial among them."""
import numpy as np
import pytest

from dispatch import stream_bytes, stream_chunks, streams_dI
from gpu_helpers import driven_current, log, np_, random_params, to_dev
from paper_2311_11390_amd.synth import rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,N,TR,dI", [(64, 1917, 256, 40, False), (4, 2877, 2048, 20, False),
                                         (8, 5980, 1000, 50, True), (16, 2350, 1024, 100, True)])
def test_noalloc_takes_the_same_chunks(B, T, N, TR, dI):
    import torch

    from paper_2311_11390_amd import alif
    assert stream_bytes(B, N, stream_chunks(B, T, N, TR)) > 12 << 20
    assert not dI or streams_dI(B, T, N, TR)
    log(f"[noalloc chunks] B={B} T={T} N={N} T_R={TR} dL/dI {dI}")
    prm = random_params(700 + TR, N, tm=(2.0, 30.0), bias=(-0.2, 0.2))
    P = to_dev(prm)
    It = torch.as_tensor(driven_current(700 + TR, B, T, N), device="cuda")
    f = alif.forward(It, P, 2.0 / TR, 2.0, save=True)
    gS = torch.as_tensor(rng(701).standard_normal((B, T, N)).astype(np.float32), device="cuda")
    ref = alif.backward(f, It, P, grad_spikes=gS, want_grad_current=dI)
    got = alif.backward(f, It, P, grad_spikes=gS, want_grad_current=dI, noalloc=True)
    torch.cuda.synchronize()
    assert int(f["spikes"].sum()) > 0
    for k, v in ref.items():
        if v is not None:
            np.testing.assert_array_equal(np_(v), np_(got[k]), err_msg=k)
