"""Device memory of finished requests kept by the server: results in kept blocks equal those
of a fresh server (also where a block is larger than the request, or held another's data),
everything held stays within the budget, and it goes back to the device after a second
without requests and with the server."""
import time

import numpy as np
import pytest

from gpu_helpers import log, random_params

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _torch_first():
    import torch
    torch.cuda.init()


def _request(N, T, seed):
    from paper_2311_11390_amd.serving import Request
    prm = random_params(seed, N, tm=(10.0, 30.0), ta=(100.0, 300.0), d=(0.0, 1.8), th=(0.9, 1.1))
    return Request(T=T, dt=0.1, arp=2.0, tau_mem=prm.tau_mem, tau_adapt=prm.tau_adapt, d=prm.d, theta0=prm.theta0,
                   seed=seed, want_spikes=True, events_capacity=N * 40)


def _free():
    import torch
    return torch.cuda.mem_get_info()[0]


def test_kept_blocks_give_the_same_results():
    from paper_2311_11390_amd import serving
    reqs = [_request(*a) for a in ((300, 4000, 1), (280, 4000, 2), (300, 4000, 3), (64, 500, 4), (299, 4000, 5),
                                   (300, 4000, 1), (500, 3000, 6), (64, 500, 4))]
    alone = []
    for r in reqs:
        with serving.Server(1 << 30, max_slots=1) as srv:
            alone.append(srv.wait(srv.submit(r)))
    for budget in (max(serving.footprint(r) for r in reqs), 1 << 30):   # one at a time; room to keep
        log(f"[serving memory] budget {budget}")
        with serving.Server(budget, max_slots=3) as srv:
            for _ in range(2):
                got = [srv.wait(t) for t in [srv.submit(r) for r in reqs]]
                for g, w in zip(got, alone):
                    assert g.status == 0 and g.n_spikes == w.n_spikes and g.n_spikes > 0
                    np.testing.assert_array_equal(g.spikes, w.spikes)
                    np.testing.assert_array_equal(g.events, w.events)


def test_held_memory_is_bounded_and_given_back():
    from paper_2311_11390_amd import serving
    reqs = [_request(1000, T, T) for T in (6000, 7000, 8000, 9000, 10000)]
    budget = int(1.2 * serving.footprint(reqs[-1]))
    slack = 32 << 20
    with serving.Server(1 << 20, max_slots=1) as srv:   # (whatever the first use of the device takes)
        srv.wait(srv.submit(_request(16, 100, 1)))
    before = _free()
    with serving.Server(budget, max_slots=2) as srv:
        least = before
        for r in reqs + reqs[::-1]:
            assert srv.wait(srv.submit(r)).status == 0
            least = min(least, _free())
        log(f"[serving memory] held {before - least} of {budget}")
        assert before - least <= budget + slack
        assert before - least >= serving.footprint(reqs[-1]) // 2
        end = time.monotonic() + 10.0
        while _free() < before - slack and time.monotonic() < end:
            time.sleep(0.1)
        assert _free() >= before - slack
        assert srv.wait(srv.submit(reqs[0])).status == 0
    assert _free() >= before - slack
