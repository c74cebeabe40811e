"""The number of time chunks of the streaming backward (a host rule, no GPU): the chunks'
sums fit the static scratch of alif_backward_noalloc, so a call takes as many with either
scratch; every chunk holds a block; and the SIMDs get whole rounds of waves."""
import pytest

from dispatch import stream_bytes, stream_chunks

SCRATCH, SIMDS = 16 << 20, 1024


@pytest.mark.parametrize("TR", [2, 20, 40, 100])
def test_chunks_fit_the_static_scratch(TR):
    for B in (1, 4, 64, 100, 128, 1000):
        for N in (1, 64, 100, 256, 1000, 2048, 20000):
            for T in (1, 100, 300, 2000, 20000):
                c = stream_chunks(B, T, N, TR)
                what = f"{B} x {N} x {T}: {c} chunks"
                waves, blocks = B * ((N + 63) // 64), -(-T // TR)
                assert 1 <= c <= min(64, blocks), what
                if c > 1:
                    assert stream_bytes(B, N, c) <= SCRATCH, what
                    assert c * waves <= 4 * SIMDS, what
                    assert -(-blocks // -(-blocks // c)) == c, what


@pytest.mark.parametrize("B,T,N,TR", [(64, 20000, 256, 40), (4, 20000, 2048, 20), (19, 13195, 773, 64),
                                      (119, 2008, 77, 120), (30, 9000, 500, 80), (10, 12000, 1001, 31)])
def test_chunks_use_the_rounds_they_take(B, T, N, TR):
    """No other count that fits gives a SIMD as many waves of shorter chunks."""
    waves, blocks = B * ((N + 63) // 64), -(-T // TR)
    c = stream_chunks(B, T, N, TR)
    rounds, longest = -(-c * waves // SIMDS), -(-blocks // c)
    for k in range(c + 1, min(64, blocks) + 1):
        if stream_bytes(B, N, k) <= SCRATCH and -(-k * waves // SIMDS) == rounds:
            assert -(-blocks // k) >= longest, f"{k} instead of {c} chunks"


def test_full_size_fits_keep_their_chunks():
    """The two fits the kernel's figures are quoted on."""
    assert stream_chunks(64, 20000, 256, 40) == 12
    assert stream_chunks(4, 20000, 2048, 20) == 24
