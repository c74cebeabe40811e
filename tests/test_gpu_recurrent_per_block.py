"""The recurrent layer over 256 neurons (a launch a block) without traces, where each
block's forward is a call of one block on a sub-range of the tensors: spikes, whole
current and carries are the bits of the same layer with traces, whose blocks run the
block kernel. Ragged last blocks, neuron tails, delays of T_R and longer."""
import numpy as np
import pytest

from dispatch import forward_chains
from gpu_helpers import driven_current, log, np_, random_params, to_dev
from paper_2311_11390_amd.synth import normal_weights

pytestmark = pytest.mark.gpu


def _carries(buf, B, NB, N):
    """The written parts of a carry buffer: v, a (float), spike step (u8), 256-byte aligned."""
    rows, out, o = B * (NB + 1) * N, [], 0
    for size in (4, 4, 1):
        out.append(buf[o:o + rows * size])
        o += -(-rows * size // 256) * 256
    return out


@pytest.mark.parametrize("TR", [2, 3, 4, 5, 8, 16, 23, 32])
@pytest.mark.parametrize("delay,sdt", [(0, 0), (3, 1)])
def test_blocks_without_traces_equal_the_traced_layer(TR, delay, sdt):
    import torch

    from paper_2311_11390_amd import alif
    from paper_2311_11390_amd.synth import rng
    B, N, dt, T = 2, 300, 2.0 / TR, 9 * TR + TR // 2 + 1
    NB = -(-T // TR)
    assert forward_chains(B, N, TR, 1, carries=True) == (TR != 3)
    assert not forward_chains(B, N, TR, 1, traces=True, carries=True)
    D = TR + delay if delay else 0
    log(f"[recurrent per block] T_R={TR} delay={D} spike dtype {sdt}")
    P = to_dev(random_params(600 + TR, N, tm=(2.0, 30.0), bias=(-0.2, 0.2)))
    I = torch.as_tensor(driven_current(600 + TR, B, T, N), device="cuda")
    Wr = torch.as_tensor(normal_weights(rng(601), N, N) * 2.0, device="cuda")
    kw = dict(delay=D, spike_dtype=sdt)
    a = alif.forward_recurrent(I, P, dt, 2.0, Wr, **kw)
    b = alif.forward_recurrent(I, P, dt, 2.0, Wr, want_v=True, want_theta=True, **kw)
    torch.cuda.synchronize()
    assert float(a["spikes"].float().sum()) > 0 and not torch.equal(a["current"], I)
    assert torch.equal(a["spikes"], b["spikes"]) and torch.equal(a["current"], b["current"])
    for x, y in zip(_carries(np_(a["carries"]), B, NB, N), _carries(np_(b["carries"]), B, NB, N)):
        np.testing.assert_array_equal(x, y)
