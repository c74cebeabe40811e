"""The recurrent layer in slices where many spikes land in a block (T_R 2-6, neurons that fire
whenever they can), recurrent sums in registers and in LDS, against the one-launch form that
calls with traces take: spikes and whole current bit for bit. Delays that reach two source
blocks and one, ragged last blocks, neuron tails."""
import pytest

from gpu_helpers import log, random_params, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("TR,delay,N", [(2, 0, 128), (2, 3, 256), (2, 0, 100), (3, 0, 128), (3, 5, 72), (4, 0, 128),
                                        (4, 6, 100), (4, 0, 256), (6, 0, 64), (6, 7, 200)])
def test_dense_slices_equal_one_launch(TR, delay, N):
    import torch

    from paper_2311_11390_amd import alif
    B, dt, T = 6, 2.0 / TR, 560000 // N // TR * TR + TR // 2
    log(f"[slices dense] T_R={TR} D={delay} T={T} N={N}")
    g = torch.Generator(device="cuda").manual_seed(TR + N)
    P = to_dev(random_params(TR + N, N, tm=(2.0, 30.0), d=(0.0, 0.02)))
    x = torch.rand(B, T, N, generator=g, device="cuda") * 8.0
    Wrec = torch.randn(N, N, generator=g, device="cuda") * (2.0 / N ** 0.5)
    a = alif.forward_recurrent(x, P, dt, 2.0, Wrec, delay=delay)
    b = alif.forward_recurrent(x, P, dt, 2.0, Wrec, delay=delay, want_v=True, want_theta=True)
    torch.cuda.synchronize()
    assert a["spikes"].float().mean() > 0.2 / TR
    assert torch.equal(a["spikes"], b["spikes"]) and torch.equal(a["current"], b["current"])
