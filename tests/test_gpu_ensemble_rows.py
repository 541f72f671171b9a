"""A band height given for an ensemble is the height of all its bands: as many
work items as those bands have tiles, and a workspace of the queried size."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(2600, 900), (130, 70), (59, 201), (181, 600)]


@pytest.mark.parametrize("rows", [1, 7, 16, 64, 4096])
def test_given_rows_are_the_band_height(rows):
    from paper_1912_02457_amd import Domain, Ensemble
    from workloads import random_small
    doms = [Domain.from_workload(random_small(nx, ny, seed=k, land_frac=0.2)) for k, (nx, ny) in enumerate(SIZES)]
    print(rows, flush=True)
    with Ensemble(doms, rows_per_wave=rows) as e:
        by, chunk, items, blocks = e.info()
        assert by == rows and items == sum(-(-nx // 60) * -(-ny // rows) for nx, ny in SIZES)
        e.step(3)
        got = [d.read_state() for d in doms]
    for k, ((nx, ny), g) in enumerate(zip(SIZES, got)):
        d = Domain.from_workload(random_small(nx, ny, seed=k, land_frac=0.2))
        d.step(3)
        assert all(np.array_equal(a, b) for a, b in zip(g, d.read_state()))
        d.close()
    for d in doms:
        d.close()
