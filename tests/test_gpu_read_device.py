"""Reading a state into device memory: widths and heights around the read's
128 columns and 8 rows, planes that start unaligned, single planes, planes that
overlap one another, pinned host memory, and the time and next step with them;
bitwise what was set."""

import ctypes as C

import numpy as np
import pytest

from test_gpu_read_staging import _domain

pytestmark = pytest.mark.gpu


def _read(dom, *ptrs):
    from paper_1912_02457_amd import swe
    t, dt = C.c_double(), C.c_double()
    swe._check(swe.load_library().swe_read_state(dom._h, *ptrs, C.byref(t), C.byref(dt)))
    return t.value, dt.value


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 9), (127, 7), (128, 8), (129, 16), (255, 17), (257, 2), (1001, 333)])
def test_read_into_device(nx, ny):
    import torch
    print(nx, ny, flush=True)
    dom, q = _domain(nx, ny, nx + ny)
    dom.step(3)
    *q, t, dt = dom.read_state()
    n = nx * ny
    big = torch.full((3 * n + 8,), -7.0, device="cuda")
    p = big.data_ptr()
    assert _read(dom, p + 4, p + 4 * (n + 2), p + 4 * (2 * n + 7)) == (t, dt)  # odd starts, gaps between
    h = big.cpu().numpy()
    for a, b in zip((1, n + 2, 2 * n + 7), q):
        assert np.array_equal(h[a:a + n].reshape(ny, nx), b)
    gaps = [0, n + 1, *range(2 * n + 2, 2 * n + 7), 3 * n + 7]
    assert (h[gaps] == -7.0).all()
    big.fill_(-7.0)
    assert _read(dom, None, p, None) == (t, dt)
    h = big.cpu().numpy()
    assert np.array_equal(h[:n].reshape(ny, nx), q[1]) and (h[n:] == -7.0).all()
    assert _read(dom, p, p + 4, p) == (t, dt)  # overlapping: written in order
    assert np.array_equal(big.cpu().numpy()[:n].reshape(ny, nx), q[2])
    pinned = torch.empty((ny, nx), pin_memory=True)
    assert _read(dom, p, pinned.data_ptr(), None) == (t, dt)
    assert np.array_equal(pinned.numpy(), q[1]) and np.array_equal(big.cpu().numpy()[:n].reshape(ny, nx), q[0])
    dom.close()
