"""Forcing tables of every length the snapshot search treats differently (one
entry, one load of 64 entries, several passes), at times before, on, between
and after the entries: nested sides and gridded wind against the oracle."""

import numpy as np
import pytest

from _parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 62, 63, 64, 65, 127, 3969, 3970])
def test_snapshot_search(n):
    from oracle import oracle as orc
    from paper_1912_02457_amd import Domain
    from workloads import BC_NESTED, BC_WALL, random_small

    rng = np.random.default_rng(n)
    wl = random_small(70, 24, seed=5, bc=(BC_NESTED, BC_WALL, BC_WALL, BC_NESTED), wind=(0.1, 0.05))
    times = 100.0 + np.cumsum(rng.uniform(1.0, 9.0, n))
    bnd = (0.3 * rng.standard_normal((n, 3, 1)) * np.ones((1, 1, wl.bnd.shape[2]))).astype(np.float32)
    w10 = (8.0 + rng.standard_normal((n, 3, 4, 2))).astype(np.float32)
    wl = wl.copy(bnd_t=times, bnd=bnd, w10_t=times + 2.5, w10=w10)
    dom = Domain.from_workload(wl)
    o = orc.Oracle(wl)
    at = [0.0, times[0], times[-1], times[-1] + 50.0]
    at += [times[k] for k in (1, n // 2, n - 2) if 0 <= k < n] + list(rng.uniform(times[0], times[-1] + 1.0, 3))
    for t0 in at:
        print("snapshots", n, "t", t0, flush=True)
        dom.set_state(wl.eta, wl.hu, wl.hv, t0)
        dom.step(3)
        got = dom.read_state()
        ref, t, _, _ = o.run(t=t0, nsteps=3)
        assert_parity(got, ref, wl.land, label=f"n={n} t0={t0}")
        assert abs(got[3] - t) <= 1e-6 * t
    dom.close()
