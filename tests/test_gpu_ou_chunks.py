"""The device OU current around the edges of its chunks of 256 steps and their parts of 32, and
of its groups of 64 neurons, against the oracle's generator: the floats agree to one ulp
(the FP64 values differ in their last bits, so a float next to a rounding boundary may too)."""
import numpy as np
import pytest

from gpu_helpers import log
from oracle import ou_philox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 31, 32, 33, 255, 256, 257, 288, 512, 545])
@pytest.mark.parametrize("N", [1, 64, 65])
def test_ou_chunk_edges(T, N):
    import torch

    from paper_2311_11390_amd import alif
    log(f"[ou] T={T} N={N}")
    got = alif.ou_current(T, N, 0.1, 3.0, 0.4, 0.7, 99 + T)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    want, want64 = ou_philox.ou_current(T, N, 0.1, 3.0, 0.4, 0.7, 99 + T)
    assert np.abs(got - want64).max() < 1e-6
    assert (np.abs(got - want) <= np.spacing(np.abs(want))).all()
