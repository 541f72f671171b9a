"""Ensembles whose bands the launch model chooses: few tiny members to many,
workspaces from the query's size down to the smallest accepted one (one band
height), and items that do not fill the last wavefront or block; every member
bitwise the domain stepped on its own."""

import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _members(sizes, comp):
    from paper_1912_02457_amd import Domain
    from workloads import random_small
    return [Domain.from_workload(random_small(nx, ny, seed=k, land_frac=0.2, wind=(0.1, 0.0)), compensated_state=comp)
            for k, (nx, ny) in enumerate(sizes)]


SIZES = {
    "one": [(61, 5)],
    "small": [(130, 70), (59, 201), (300, 40)],
    "mixed": [(2, 2), (700, 333), (64, 64), (181, 600), (1000, 3)],
    "many": [(40 + 7 * k, 90 - 3 * k) for k in range(25)],
}


@pytest.mark.parametrize("comp", [True, False])
@pytest.mark.parametrize("chunk", [0, 3, 64])
@pytest.mark.parametrize("which", list(SIZES))
def test_bands_leave_members_alone(which, chunk, comp):
    from paper_1912_02457_amd import Ensemble
    a, b = _members(SIZES[which], comp), _members(SIZES[which], comp)
    print(which, chunk, comp, flush=True)
    with Ensemble(a, chunk=chunk) as e:
        e.step(9)
        for d in b:
            d.step(9)
        for x, y in zip(a, b):
            p, q = x.read_state(), y.read_state()
            assert all(np.array_equal(s, t) for s, t in zip(p[:3], q[:3])) and p[3:] == q[3:]
    for d in a + b:
        d.close()


@pytest.mark.parametrize("which", ["small", "mixed"])
def test_smallest_accepted_workspace(which):
    import torch
    from paper_1912_02457_amd import swe
    L = swe.load_library()
    a, b = _members(SIZES[which], True), _members(SIZES[which], True)
    arr = (C.c_void_p * len(a))(*[d._h for d in a])
    n = C.c_size_t()
    swe._check(L.swe_ensemble_workspace_bytes(arr, len(a), 0, C.byref(n)))
    ws = torch.zeros(n.value, dtype=torch.uint8, device="cuda")

    def create(nbytes):
        h = C.c_void_p()
        rc = L.swe_ensemble_create(arr, len(a), C.c_void_p(ws.data_ptr()), nbytes, None, 0, 0, C.byref(h))
        return rc, h

    lo, hi = 0, n.value  # refused, accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        rc, h = create(mid)
        if rc == swe.SWE_OK:
            L.swe_ensemble_destroy(h)
            hi = mid
        else:
            assert rc == swe.SWE_E_NOMEM
            lo = mid
    assert hi < n.value  # the query asks for more items than one height of 16 rows gives
    rc, h = create(hi)
    assert rc == swe.SWE_OK
    swe._check(L.swe_ensemble_step(h, 5))
    torch.cuda.synchronize()
    L.swe_ensemble_destroy(h)
    for d in b:
        d.step(5)
    for x, y in zip(a, b):
        p, q = x.read_state(), y.read_state()
        assert all(np.array_equal(s, t) for s, t in zip(p[:3], q[:3])) and p[3:] == q[3:]
    for d in a + b:
        d.close()
