"""The straight-line variants of a row's fluxes (deep water, deep water beside
land, everything else) and the relaxation-zone tables of a tile: rows that mix
water around the depth where the wet-dry treatment starts, dry ground and land,
in bands lower and taller than the 64 rows a zone table holds.  Every tiling
gives the same bits, and the result is the oracle's."""

import numpy as np
import pytest

from _parity import assert_parity

pytestmark = pytest.mark.gpu

DEEP = 1.0 / 64.0  # kappa = 1e-3: deep_water() of csrc/swe_device.h


def _workload(kind, nested, frs_width):
    from workloads import BC_NESTED, BC_WALL, random_small
    land = 0.15 if "land" in kind else 0.0
    wl = random_small(131, 150, seed=11, bc=(BC_NESTED,) * 4 if nested else (BC_WALL,) * 4, land_frac=land,
                      wet_dry="dry" in kind, wind=(0.1, -0.05))
    wl = wl.copy(frs_width=frs_width)
    if "shallow" in kind:
        # a sill whose depth runs from half to twice the threshold, at rest
        Hc = wl.Hc.copy()
        x = np.linspace(0.5, 2.0, 40)
        Hc[60:80, 40:80] = (DEEP * x)[None, :]
        eta, hu, hv = (a.copy() for a in (wl.eta, wl.hu, wl.hv))
        for a in (eta, hu, hv):
            a[58:82, 38:82] = 0.0
        wl = wl.copy(Hc=Hc.astype(np.float32), eta=eta, hu=hu, hv=hv)
    return wl


@pytest.mark.parametrize("nested,frs_width", [(False, 10), (True, 10), (True, 32)])
@pytest.mark.parametrize("kind", ["deep", "shallow", "dry", "land", "land dry shallow"])
def test_row_variants(kind, nested, frs_width):
    from oracle import oracle as orc
    from paper_1912_02457_amd import Domain

    wl = _workload(kind, nested, frs_width)
    ref, _, dts, _ = orc.Oracle(wl).run(nsteps=8)
    for comp in (True, False):
        first = None
        for rows in (3, 64, 65, 150):
            print(kind, nested, frs_width, comp, rows, flush=True)
            dom = Domain.from_workload(wl, compensated_state=comp)
            dom.set_tiling(rows)
            dom.step_dt(dts)
            got = dom.read_state()
            dom.close()
            if first is None:
                first = got
                assert_parity(got, ref, wl.land, label=f"{kind} {nested} {frs_width} {comp}")
            for a, b in zip(got[:3], first[:3]):
                assert np.array_equal(a, b), f"{rows} rows differ"
