"""The tiling tuner starts from what the domain has: the tiling in use and the
built-in choice are among the tilings it may time, so that tuning cannot end
on something slower than either.  (A height of one row is listed as two-row
bands with every row in a one-row tail, which is the same work.)"""

import numpy as np
import pytest
import torch  # noqa: F401  (its GPU runtime first)

pytestmark = pytest.mark.gpu


def _form(t, ny):
    return (2, 1, ny) if t[:3] == (1, 0, 0) else t[:3]


@pytest.mark.parametrize("nx,ny,comp", [(133, 71, True), (300, 200, False), (777, 333, True), (2048, 2048, True),
                                        (3, 2, False)])
def test_default_and_current_tilings_are_candidates(nx, ny, comp):
    from paper_1912_02457_amd import Domain
    from workloads import random_small
    wl = random_small(nx, ny, seed=5, land_frac=0.1)
    d = Domain.from_workload(wl, compensated_state=comp)
    print(nx, ny, comp, d.stage_tiling(1), d.stage_tiling(2), flush=True)
    for stage in (1, 2):
        built_in = _form(d.stage_tiling(stage), ny)
        assert built_in in d.list_tilings(stage)
        d.set_stage_tiling(stage, 11, 4, min(9, ny - 1))
        got = d.list_tilings(stage)
        assert d.stage_tiling(stage)[:3] in got and built_in in got
        assert len(set(got)) == len(got)
        # every entry can be set, and is reported as it is listed
        for t in got:
            d.set_stage_tiling(stage, *t)
            assert d.stage_tiling(stage)[:3] == t
    d.set_tiling(0)
    ref = Domain.from_workload(wl, compensated_state=comp)
    d.autotune()
    for stage in (1, 2):
        assert d.stage_tiling(stage)[:3] in d.list_tilings(stage)
    # one-row bands in either form, and the tuned tiling, give the same state
    for t in ((2, 1, ny), (1, 0, 0)):
        e = Domain.from_workload(wl, compensated_state=comp)
        for stage in (1, 2):
            e.set_stage_tiling(stage, *t)
        assert e.stage_tiling(1)[4] == e.stage_tiling(2)[4] == -(-nx // 60) * ny
        e.step(11)
        ref2 = e.read_state()
        e.close()
    d.step(11)
    ref.step(11)
    for a, b, c in zip(d.read_state(), ref.read_state(), ref2):
        assert np.array_equal(a, b) and np.array_equal(a, c)
    d.close()
    ref.close()
