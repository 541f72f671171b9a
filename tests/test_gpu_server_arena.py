"""An arena that holds N requests and the work lists of one band height holds
them all at once: what the server takes beyond that for shorter bands is given
back when a request needs the room, also while steps that use it are queued."""

import numpy as np
import pytest
import torch  # noqa: F401  (its GPU runtime first)

pytestmark = pytest.mark.gpu

N = 6
SLACK = 768 << 10  # the lists of 16-row bands (110 KiB for all six, twice while one grows) and the holes they leave


def _request(k):
    from workloads import config5_member
    return config5_member(2000, 800, 0)


def _run(n, slack, waves):
    """Submits by waves with a tick after each, all active at once; returns the
    arena bytes in use beyond the requests' own after each wave's tick."""
    from paper_1912_02457_amd import Domain, Server, workspace_bytes
    from paper_1912_02457_amd.swe import params_of
    wl = _request(0)
    one = (workspace_bytes(params_of(wl), 1, 0) + 255) // 256 * 256
    print(n, slack, waves, one, flush=True)
    extra = []
    with Server(n * one + slack, max_active=16, steps_per_tick=4) as srv:
        sent, horizon = 0, 100.0
        for w in waves:
            for _ in range(w):
                srv.submit(wl, horizon, req_id=sent)
                sent += 1
            active, waiting = srv.tick()
            assert (active, waiting) == (sent, 0)
            extra.append(srv.stats()["arena_used"] - sent * one)
        done = []
        for _ in range(200):
            active, waiting = srv.tick()
            done += srv.poll()
            if active == 0 and waiting == 0:
                break
        st = srv.stats()
    assert sorted(c["id"] for c in done) == list(range(n))
    assert st["arena_used"] == 0 and st["arena_peak"] <= n * one + slack
    d = Domain.from_workload(wl)
    steps = d.run_until(horizon)
    ref = d.read_state()
    d.close()
    for c in done:
        assert c["status"] == 0 and c["steps"] == steps and c["t"] == ref[3]
        assert all(np.array_equal(a, b) for a, b in zip(c["state"], ref[:3]))
    return extra


@pytest.mark.parametrize("waves", [[6], [5, 1], [1, 1, 1, 1, 1, 1], [3, 0, 3]])
def test_arena_for_n_requests_holds_n(waves):
    _run(N, SLACK, waves)


def test_spare_block_in_use_is_given_back_for_a_request():
    # one request: a list of 16-row bands (14 KiB, 22 taken) and beside it one of
    # the chosen bands (33 KiB), which leaves no room for the list of two (28
    # KiB)
    extra = _run(2, 72 << 10, [1, 0, 1])
    assert extra[0] < 24 << 10 and extra[1] > 48 << 10 and extra[2] > 56 << 10
