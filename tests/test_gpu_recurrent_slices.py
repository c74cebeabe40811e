"""The recurrent layer run in several slices of blocks (runs that expand to 90 MB and
more) against the one-launch form that calls with traces take: the same arithmetic in the
same order, so spikes, whole current and carries agree bit for bit. Delays of one block, of
several and not a whole number of blocks; a ragged last block; four neurons a lane and one
(N % 4 != 0, a misaligned output); a current that lies in place (spike input); the three
spike types."""
import pytest

from gpu_helpers import log, random_params, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("TR,delay,T,N,sdt,spikes_in", [
    (10, 0, 6003, 256, 0, False), (10, 37, 6003, 255, 1, False), (40, 0, 6000, 256, 2, False),
    (2, 5, 6001, 130, 0, True), (40, 80, 6017, 200, 0, True), (47, 50, 6100, 128, 1, False),
    (10, 0, 1003, 256, 0, False), (20, 30, 801, 255, 1, False), (40, 0, 900, 128, 2, True)])   # (one launch)
def test_slices_equal_one_launch(TR, delay, T, N, sdt, spikes_in):
    import torch

    from paper_2311_11390_amd import alif
    B, dt, n_in = 10, 2.0 / TR, 12
    log(f"[slices] T_R={TR} D={delay} T={T} N={N} spike type {sdt} spike input {spikes_in}")
    g = torch.Generator(device="cuda").manual_seed(TR + N)
    P = to_dev(random_params(TR, N, tm=(2.0, 30.0), d=(0.0, 0.5)))
    if spikes_in:
        x = (torch.rand(B, T, n_in, generator=g, device="cuda") < 0.3).to(torch.uint8)
        W = torch.randn(N, n_in, generator=g, device="cuda") + 0.4
    else:
        x = torch.randn(B, T, N, generator=g, device="cuda") * 3.0 + 1.5  # (noise alone averages out at fine steps)
        W = None
    Wrec = torch.randn(N, N, generator=g, device="cuda") * 0.3
    a = alif.forward_recurrent(x, P, dt, 2.0, Wrec, W, spike_dtype=sdt, delay=delay)
    b = alif.forward_recurrent(x, P, dt, 2.0, Wrec, W, spike_dtype=sdt, delay=delay, want_v=True, want_theta=True)
    torch.cuda.synchronize()
    assert a["spikes"].float().sum() > 1000
    for k in ("spikes", "current", "carries"):
        if k == "carries":   # (256-byte alignment gaps between the planes are never written)
            NB, n = (T + TR - 1) // TR, B * ((T + TR - 1) // TR + 1) * N
            up = lambda v: (v + 255) // 256 * 256
            for off, size in ((0, 4 * n), (up(4 * n), 4 * n), (2 * up(4 * n), n)):
                assert torch.equal(a[k][off:off + size], b[k][off:off + size]), (k, off)
        else:
            assert torch.equal(a[k], b[k]), k
