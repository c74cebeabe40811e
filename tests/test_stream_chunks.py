"""The number of time chunks of the streaming backward (a host rule, no GPU): the chunks'
sums fit the static scratch of alif_backward_noalloc, so a call takes as many with either
scratch, and no fewer than that scratch or the waves aimed at allow."""
import pytest

from dispatch import stream_bytes, stream_chunks

SCRATCH = 16 << 20


@pytest.mark.parametrize("TR", [2, 20, 40, 100])
def test_chunks_fit_the_static_scratch(TR):
    for B in (1, 4, 64, 100, 128, 1000):
        for N in (1, 64, 100, 256, 1000, 2048, 20000):
            for T in (1, 100, 2000, 20000):
                c = stream_chunks(B, T, N, TR)
                what = f"{B} x {N} x {T}: {c} chunks"
                assert c >= 1, what
                if c > 1:
                    assert stream_bytes(B, N, c) <= SCRATCH, what
                waves = B * ((N + 63) // 64)
                blocks = -(-T // TR)
                want = min(-(-3072 // waves), T // 64, blocks, 64)
                most = min(want, SCRATCH // (stream_bytes(B, N, 2) // 2))
                if most > 1:   # as many as the blocks split into evenly
                    assert c == -(-blocks // -(-blocks // most)), what


def test_full_size_fits_keep_their_chunks():
    """The two fits the kernel's figures are quoted on."""
    assert stream_chunks(64, 20000, 256, 40) == 12
    assert stream_chunks(4, 20000, 2048, 20) == 24
