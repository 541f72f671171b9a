"""The launch model (csrc/swe_tiling.h) on the host: exact against a plain
simulation of every CU where the order among CUs does not matter, never below
the bound that skips candidates, within a block of the simulation elsewhere,
and without memory allocations (it runs inside calls that promise none)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1912_02457_amd", "csrc")
ROCM_INCLUDE = "/opt/rocm/include"

CHECK = r"""
#include "swe_tiling.h"
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>
#include <vector>
using namespace swe;

static long allocations = 0;
void *operator new(std::size_t n) { ++allocations; void *p = std::malloc(n); if (!p) std::abort(); return p; }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

// every CU on its own; CUs that have room at the same time are served in turn,
// one block each
static double plain(long n1, double c1, long n2, double c2, int ncu, int room)
{
    std::vector<std::vector<double>> cu(ncu);
    std::vector<double> since(ncu, 0.0);
    auto take = [&](double &c) { if (n1 > 0) { --n1; c = c1; return true; } if (n2 > 0) { --n2; c = c2; return true; } return false; };
    auto pace = [](size_t n) { return 1.0 / (1.0 + kSharing * ((double)n - 1)); };
    double c, last = 0.0;
    std::vector<int> open;
    for (int q = 0; q < ncu; ++q) open.push_back(q);
    while (true) {
        for (bool more = true; more;) {
            more = false;
            for (int q : open) if ((int)cu[q].size() < room && take(c)) { cu[q].push_back(c); more = true; }
        }
        double t = 1e300;
        auto end = [&](int q) { return since[q] + *std::min_element(cu[q].begin(), cu[q].end()) / pace(cu[q].size()); };
        for (int q = 0; q < ncu; ++q) if (!cu[q].empty()) t = std::min(t, end(q));
        if (t == 1e300) return last;
        last = t;
        open.clear();
        for (int q = 0; q < ncu; ++q) if (!cu[q].empty() && end(q) < t + 1e-9) {
            open.push_back(q);
            std::vector<double> y;
            const double done = (t - since[q]) * pace(cu[q].size());
            for (double w : cu[q]) if (w - done > 1e-9) y.push_back(w - done);
            cu[q] = y; since[q] = t;
        }
    }
}

int main()
{
    long bad = 0, cases = 0, exact = 0;
    auto check = [&](long n1, double c1, long n2, double c2, int ncu, int room) {
        if (n1 + n2 == 0) return;
        ++cases;
        const double a = launch_rows(n1, c1, n2, c2, ncu, room), least = launch_rows_least(n1, c1, n2, c2, ncu, room);
        const double b = plain(n1, c1, n2, c2, ncu, room);
        // one CU, or one round of equal blocks: nothing depends on which of two
        // CUs is served first
        const bool alike = ncu == 1 || (n1 + n2 <= (long)ncu * room && (n1 == 0 || n2 == 0 || c1 == c2));
        exact += alike;
        const double tol = alike ? 1e-9 * b : c2 * (1.0 + kSharing * (room - 1)) + 1e-9 * b;
        if (!(std::abs(a - b) <= tol) || !(a > 0.0) || least > a * (1 + 1e-12)) {
            if (++bad < 10) printf("n %ld %ld c %g %g ncu %d room %d: %.9g plain %.9g least %.9g\n", n1, n2, c1, c2, ncu, room, a, b, least);
        }
    };
    std::mt19937 r(11);
    for (int ncu : {1, 2, 3, 7}) for (int room = 1; room <= 8; ++room)
        for (long n1 : {0L, 1L, 2L, 5L, 22L, 61L}) for (long n2 : {0L, 1L, 3L, 9L, 40L}) {
            check(n1, 7.5, n2, 3.5, ncu, room);
            check(n1, 2.5, n2, 2.5, ncu, room);
        }
    for (int k = 0; k < 1500; ++k) {
        const double c1 = 2.5 + r() % 15, c2 = 2.5 + r() % 4;
        check(r() % 2000, std::max(c1, c2), r() % 2000, std::min(c1, c2), 1 + r() % 40, 1 + r() % 8);
    }
    // both stages at once: each what it would be alone
    for (int w1 = 1; w1 <= 8; ++w1) for (int w2 = 1; w2 <= 8; ++w2) for (int nx : {61, 777, 2600}) {
        const int w[2] = {w1, w2};
        Tiling T[2];
        default_tilings(nx, 333, 256, w, T);
        for (int q = 0; q < 2; ++q) {
            const Tiling U = default_tiling(nx, 333, 256, w[q]);
            bad += T[q].by != U.by || T[q].by2 != U.by2 || T[q].nrb1 != U.nrb1 || T[q].nblocks != U.nblocks || T[q].order != U.order;
        }
    }
    const std::pair<int, int> one[] = {{777, 333}}, many[] = {{2600, 900}, {61, 1}, {300, 200}, {1000, 600}};
    const long before = allocations;
    for (int w = 1; w <= 8; ++w) for (int nx : {2, 128, 2600, 30000}) bad += default_tiling(nx, 900, 256, w).by < 1;
    bad += ensemble_bands(one, 0, 256).by < 1;
    bad += ensemble_bands(many, 0, 256).by < 1;
    if (allocations != before) { ++bad; printf("allocations: %ld\n", allocations - before); }
    printf("cases %ld exact %ld bad %ld\n", cases, exact, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                    reason="needs g++ and the HIP headers")
def test_launch_model(tmp_path):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROCM_INCLUDE}", f"-I{CSRC}", str(src), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-2500:] + r.stderr[-2000:]
