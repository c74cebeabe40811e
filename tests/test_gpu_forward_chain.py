"""The forward of layers that do not fill the card (T_R 2-32) with its chain, loads and
stores on waves of their own, against the block kernel that calls with traces take: the same operations, so
spikes, carries and final states agree bit for bit. Lengths around the groups of 2-16 blocks
and a ragged last block, neuron tails, the three spike types, runs that start from saved
states, and both sides of the size where the layer goes back to the block kernel."""
import pytest

from gpu_helpers import log, random_params, to_dev

pytestmark = pytest.mark.gpu


def _planes(c, B, T, N, TR):   # (the alignment gaps between the planes are never written)
    n, up = B * ((T + TR - 1) // TR + 1) * N, lambda v: (v + 255) // 256 * 256
    return [c[o:o + s] for o, s in ((0, 4 * n), (up(4 * n), 4 * n), (2 * up(4 * n), n))]


@pytest.mark.parametrize("TR", [2, 3, 4, 5, 6, 7, 8, 9, 10, 13, 16, 17, 20, 21, 24, 25, 31, 32])
@pytest.mark.parametrize("B,N,blocks,missing", [(1, 1, 1, 1), (1, 64, 3, 0), (2, 65, 8, 0), (3, 100, 16, 1),
                                                (2, 130, 17, 0), (1, 63, 33, 1), (2, 200, 201, 0), (10, 4096, 65, 0),
                                                (10, 4160, 65, 1), (16, 4100, 65, 1)])
def test_chain_equals_block_kernel(TR, B, N, blocks, missing):
    import torch

    from paper_2311_11390_amd import alif
    T = blocks * TR - missing
    log(f"[chain] T_R={TR} B={B} N={N} T={T}")
    g = torch.Generator(device="cuda").manual_seed(TR * 1000 + T)
    P = to_dev(random_params(TR + N, N, tm=(2.0, 30.0), d=(0.0, 0.5), bias=(-0.3, 0.3)))
    x = torch.randn(B, T, N, generator=g, device="cuda") * 3.0 + 1.5
    init = {"v": torch.rand(B, N, generator=g, device="cuda", dtype=torch.float64) * 0.3,
            "a": torch.rand(B, N, generator=g, device="cuda", dtype=torch.float64),
            "ts": torch.randint(0, TR + 1, (B, N), generator=g, device="cuda", dtype=torch.int32)}
    dt = 2.0 / TR
    for sdt, save, start in ((0, True, None), (1, False, None), (2, True, init), (0, False, init)):
        kw = dict(spike_dtype=sdt, save=save, init=start, want_final=T % TR == 0)
        a = alif.forward(x, P, dt, 2.0, **kw)
        b = alif.forward(x, P, dt, 2.0, want_v=True, **kw)
        torch.cuda.synchronize()
        assert torch.equal(a["spikes"], b["spikes"])
        assert blocks < 65 or a["spikes"].float().sum() > B * N
        for k in ("v", "a", "ts") if T % TR == 0 else ():
            assert torch.equal(a["final"][k], b["final"][k]), k
        if save:
            for p, q in zip(_planes(a["carries"], B, T, N, TR), _planes(b["carries"], B, T, N, TR)):
                assert torch.equal(p, q)
