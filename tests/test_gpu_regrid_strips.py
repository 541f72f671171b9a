"""Erosion, refinement and coarsening where their strips of columns and
segments of rows end: one column or row either side of each, fields that lie
unaligned inside larger arrays, land bytes other than 1, NaN behind land.
Masks, erosion and sampled corners are exact; refined and averaged values
take 2-4 float32 roundings of values of size max|v|: 1e-6 max|v|.  Corner
depths: 16 float32 roundings a round, 2e-5 max|Hm| as over the 11 rounds there."""

import numpy as np
import pytest

from test_gpu_preprocess import FIELD_TOL, RECON_TOL, P, _cuda, _host, swe  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(1, 9), (2, 2), (61, 4), (62, 5), (63, 3), (64, 8), (65, 1), (124, 7), (125, 13), (126, 4), (127, 2), (252, 6)]


def _inputs(nx, ny, nf):
    rng = np.random.default_rng(100 * nx + ny)
    F = rng.standard_normal((nf, ny, nx)).astype(np.float32)
    land = (rng.uniform(size=(ny, nx)) < 0.4).astype(np.uint8) * rng.integers(1, 256, (ny, nx)).astype(np.uint8)
    Hc = rng.uniform(1.0, 200.0, (ny + 1, nx + 1)).astype(np.float32)
    return F, land, Hc


def _unaligned(a):
    """The array on the device, starting one element into its allocation."""
    import torch
    flat = torch.empty(a.size + 1, dtype=torch.from_numpy(a).dtype, device="cuda")[1:]
    flat.copy_(torch.from_numpy(a).reshape(-1))
    return flat.view(a.shape)


@pytest.mark.parametrize("put", [_cuda, _unaligned])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_strip_edges(swe, nx, ny, put):  # noqa: F811
    print(nx, ny, put.__name__, flush=True)
    F, land, Hc = _inputs(nx, ny, 3)
    ref = P.erode_land(land, Hc[:-1, :-1], *F, land_depth=5.0)
    got = swe.erode_land(put(land), put(np.ascontiguousarray(Hc[:-1, :-1])), *[put(f) for f in F], land_depth=5.0)
    for r, g in zip(ref, got):
        assert np.array_equal(_host(g).astype(np.float64), np.asarray(r, np.float64))
    fo, lo, ho = swe.refine2(put(F), put(land), put(Hc), theta=1.3)
    rf, rl, rh = P.refine2(list(F), land, Hc, theta=1.3)
    assert np.abs(_host(fo) - np.stack(rf)).max() <= FIELD_TOL * np.abs(F).max()
    assert np.array_equal(_host(lo), rl != 0)  # any byte but 0 is land, masks come out as 0 or 1
    assert np.abs(_host(ho) - rh).max() <= FIELD_TOL * np.abs(Hc).max()
    only = swe.refine2(None, None, put(Hc))  # corners without a field
    assert np.array_equal(_host(only[2]), _host(ho))
    X, l2, H2 = np.repeat(np.repeat(F, 2, 1), 2, 2), lo, ho
    X = X + 0.1 * np.random.default_rng(1).standard_normal(X.shape).astype(np.float32)
    mixed = (np.random.default_rng(2).uniform(size=X.shape[1:]) < 0.5).astype(np.uint8)
    for m in (rl, mixed, None):
        cf, cl, ch = swe.coarsen2(put(X), None if m is None else put(m), H2)
        of, ol, oh = P.coarsen2(list(X), m, _host(H2))
        assert np.abs(_host(cf) - np.stack(of)).max() <= FIELD_TOL * np.abs(X).max()
        assert m is None or np.array_equal(_host(cl), ol)
        assert np.array_equal(_host(ch).astype(np.float64), oh)


@pytest.mark.parametrize("land_on", [True, False])
@pytest.mark.parametrize("nx,ny", [(57, 12), (58, 3), (59, 13), (66, 9), (67, 17), (125, 10), (183, 29), (60, 9001)])
def test_corner_depths_at_strip_edges(swe, nx, ny, land_on):  # noqa: F811
    """One strip to four, segments with and without rows outside the domain,
    the short and (last size) the long segments, odd and even rounds."""
    print(nx, ny, land_on, flush=True)
    rng = np.random.default_rng(nx + ny)
    Hm = rng.uniform(5.0, 80.0, (ny, nx)).astype(np.float32)
    land = (rng.uniform(size=(ny, nx)) < 0.3).astype(np.uint8) if land_on else None
    if land_on:
        land[:, nx // 3:nx // 3 + 6] = 200  # corners that touch no water
    for iters in (0, 1, 2, 5) if ny < 9000 else (2,):
        ref = P.reconstruct_bathymetry(Hm, None if land is None else (land != 0).astype(np.uint8), iters=iters)
        got = _host(swe.reconstruct_bathymetry(_cuda(Hm), None if land is None else _cuda(land), iters=iters))
        assert np.abs(got - ref).max() <= RECON_TOL * np.abs(Hm).max()


def test_corner_depths_of_many_segments(swe):  # noqa: F811
    """The longest segments, which only large grids take: windows of rows
    against the oracle, which reaches 3 k + 2 cells in k rounds."""
    nx, ny, k = 60, 49157, 3
    rng = np.random.default_rng(8)
    Hm = rng.uniform(5.0, 80.0, (ny, nx)).astype(np.float32)
    land = (rng.uniform(size=(ny, nx)) < 0.3).astype(np.uint8)
    print(nx, ny, k, flush=True)
    got = _host(swe.reconstruct_bathymetry(_cuda(Hm), _cuda(land), iters=k))
    for lo in (0, 1007, 24999, ny - 100):
        a, b = max(0, lo - 12), min(ny, lo + 112)
        ref = P.reconstruct_bathymetry(Hm[a:b], land[a:b], iters=k)
        end = ny + 1 if b == ny else lo + 100
        assert np.abs(got[lo:end] - ref[lo - a:end - a]).max() <= RECON_TOL * np.abs(Hm).max()


def test_land_values_stay_behind_the_mask(swe):  # noqa: F811
    """NaN and infinities on land reach no water cell."""
    nx, ny = 130, 22
    F, land, _ = _inputs(nx, ny, 2)
    bad = F.copy()
    bad[0, land != 0], bad[1, land != 0] = np.nan, np.inf
    a, b = swe.refine2(_cuda(F), _cuda(land))[0], swe.refine2(_cuda(bad), _cuda(land))[0]
    wet = np.repeat(np.repeat(land == 0, 2, 0), 2, 1)
    assert np.array_equal(_host(a)[:, wet], _host(b)[:, wet])
    one = (np.random.default_rng(5).uniform(size=(ny, nx)) < 0.4).astype(np.uint8)
    F[:, one != 0] = np.nan
    got = _host(swe.coarsen2(_cuda(F), _cuda(one))[0])
    some = (one.reshape(ny // 2, 2, nx // 2, 2) == 0).any(axis=(1, 3))
    assert np.isfinite(got[:, some]).all()
    e = _host(swe.erode_land(_cuda(one), _cuda(F[0]), _cuda(F[1]))[2])
    ref = P.erode_land(one, F[0], F[1], F[1], F[1])
    assert np.array_equal(np.isfinite(e), np.isfinite(ref[2]))
