"""Host reads of several domains by several threads run side by side: each call
copies through a staging buffer of its own.  (One after another, four threads
take four times as long as one; side by side they share the link and the
host's memory.)"""

import threading
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _domain(nx, ny, seed):
    import torch
    from paper_1912_02457_amd import Domain, make_params
    rng = np.random.default_rng(seed)
    q = [rng.uniform(-1, 1, (ny, nx)).astype(np.float32) for _ in range(3)]
    p = make_params(nx, ny, 100.0, 100.0)
    with torch.cuda.stream(torch.cuda.Stream()):
        return Domain(p, np.full((ny + 1, nx + 1), 50.0, np.float32), np.zeros((ny, nx), np.float32), *q), q


def test_reads_of_several_threads_run_side_by_side():
    doms = [_domain(1375, 664, k) for k in range(4)]

    def rounds(n):
        bad = []

        def work(d, q):
            for _ in range(10):
                got = d.read_state()
                if not all(np.array_equal(a[::97], b[::97]) for a, b in zip(got[:3], q)):
                    bad.append(d)

        best = 1e9
        for _ in range(8):
            ts = [threading.Thread(target=work, args=x) for x in doms[:n]]
            t0 = time.perf_counter()
            for t in ts:
                t.start()
            for t in ts:
                t.join()
            best = min(best, time.perf_counter() - t0)
        assert not bad
        return best

    for _ in range(3):  # a host busy with something else may spoil one attempt
        one, four = rounds(1), rounds(4)
        print(f"ten reads: {one * 1e3:.1f} ms on one thread, {four * 1e3:.1f} ms on each of four", flush=True)
        if four < 2.7 * one:
            break
    assert four < 2.7 * one
    for d, _ in doms:
        d.close()


def test_uploads_and_reads_of_several_threads():
    import torch
    bad = []

    def work(k):
        try:
            for n in range(6):
                d, q = _domain(150 + 37 * k + 211 * n, 90 + 41 * n, 10 * k + n)
                p = [a[::-1].copy() for a in q]
                ok = all(np.array_equal(a, b) for a, b in zip(d.read_state()[:3], q))
                d.set_state(*p, 5.0)
                got = d.read_state()
                ok = ok and got[3] == 5.0 and all(np.array_equal(a, b) for a, b in zip(got[:3], p))
                d.close()
                if not ok:
                    bad.append((k, n))
        except Exception as e:  # shown by the main thread
            bad.append((k, repr(e)))

    torch.cuda.synchronize()
    ts = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
