"""Reading a state into host arrays: through the staging buffer at once, in
halves (planes larger than it together, rows that do not divide it), mixed with
device tensors, from several threads, and equal to the device copy bitwise."""

import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _domain(nx, ny, seed):
    from paper_1912_02457_amd import Domain, make_params
    rng = np.random.default_rng(seed)
    q = [rng.uniform(-1, 1, (ny, nx)).astype(np.float32) for _ in range(3)]
    p = make_params(nx, ny, 100.0, 100.0)
    return Domain(p, np.full((ny + 1, nx + 1), 50.0, np.float32), np.zeros((ny, nx), np.float32), *q), q


# the last two do not fit the 64 MiB buffer: 3 planes of 22 MiB, one of 78 MiB
@pytest.mark.parametrize("nx,ny", [(2, 2), (61, 3), (1375, 664), (2401, 2402), (4600, 4431)])
def test_read_state_host_equals_device(nx, ny):
    import torch
    dom, q = _domain(nx, ny, nx)
    print(nx, ny, flush=True)
    got = dom.read_state()
    for a, b in zip(got[:3], q):
        assert np.array_equal(a, b)
    dev = [torch.empty((ny, nx), device="cuda") for _ in range(3)]
    t, dt = dom.read_state_into(*dev)
    assert (t, dt) == got[3:]
    for a, b in zip(dev, q):
        assert np.array_equal(a.cpu().numpy(), b)
    # one host array among device tensors
    from paper_1912_02457_amd import swe
    host = np.empty((ny, nx), np.float32)
    swe._check(swe.load_library().swe_read_state(dom._h, dev[0].data_ptr(), host.ctypes.data, None, None, None))
    assert np.array_equal(host, q[1]) and np.array_equal(dev[0].cpu().numpy(), q[0])
    dom.close()


def test_reads_from_several_threads():
    import torch
    doms = []
    for k in range(4):
        with torch.cuda.stream(torch.cuda.Stream()):
            doms.append(_domain(700 + 13 * k, 400, k))
    bad = []

    def work(d, q):
        for _ in range(20):
            got = d.read_state()
            if not all(np.array_equal(a, b) for a, b in zip(got[:3], q)):
                bad.append(d.nx)

    ts = [threading.Thread(target=work, args=x) for x in doms]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
    for d, _ in doms:
        d.close()
