"""The built-in tiling choice on the host (csrc/swe_tiling.h): for ragged,
narrow, tiny and large domains and every occupancy the tiling covers each
(strip, row) exactly once, stays within the heights it may choose from, and the
launch model behind it agrees with a plain event simulation of every CU."""

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
using namespace swe;

// the model, one CU at a time: first come, first served
static double plain(long n1, double c1, long n2, double c2, int ncu, int room)
{
    std::vector<std::vector<double>> cu(ncu);
    std::vector<double> since(ncu, 0.0);
    auto take = [&](double &c) { if (n1 > 0) { --n1; c = c1; return true; } if (n2 > 0) { --n2; c = c2; return true; } return false; };
    double c, last = 0.0;
    for (int l = 0; l < room; ++l) for (auto &x : cu) if ((int)x.size() == l && take(c)) x.push_back(c);
    while (true) {
        int k = -1; double t = 1e300;
        auto pace = [](size_t n) { return 1.0 / (1.0 + kSharing * ((double)n - 1)); };
        for (int q = 0; q < ncu; ++q) if (!cu[q].empty()) {
            const double e = since[q] + *std::min_element(cu[q].begin(), cu[q].end()) / pace(cu[q].size());
            if (e < t - 1e-9) { t = e; k = q; }
        }
        if (k < 0) return last;
        last = t;
        std::vector<double> y;
        const double done = (t - since[k]) * pace(cu[k].size());
        for (double w : cu[k]) if (w - done > 1e-9) y.push_back(w - done);
        while ((int)y.size() < room && take(c)) y.push_back(c);
        cu[k] = y; since[k] = t;
    }
}

int main()
{
    long bad = 0, cases = 0;
    const int nxs[] = {2, 59, 60, 61, 333, 1000, 2600, 30000}, nys[] = {2, 3, 17, 128, 501, 900, 4000};
    for (int nx : nxs) for (int ny : nys) for (int w = 1; w <= 8; ++w) {
        const Tiling T = default_tiling(nx, ny, 256, w);
        ++cases;
        std::vector<unsigned char> seen((size_t)T.nstrips * ny, 0);
        for (int b = 0; b < T.nblocks; ++b) for (int q = 0; q < kWavesPerBlock; ++q) {
            const int t = block_tile(T, b, q);
            if (t < 0) continue;
            int s, y0, y1;
            tile_place(T, t, ny, s, y0, y1);
            if (s < 0 || s >= T.nstrips || y0 < 0 || y1 > ny || y0 >= y1) { ++bad; continue; }
            for (int y = y0; y < y1; ++y) seen[(size_t)s * ny + y]++;
        }
        for (unsigned char v : seen) bad += v != 1;
        bad += T.by < 1 || T.by > 16 || T.by > ny || T.by2 < 1 || T.by2 > T.by;
    }
    // equal steps of several CUs may take their blocks in another order, so
    // the two simulations may differ by one short block at the end
    for (int ncu : {1, 3, 7}) for (int room = 1; room <= 5; ++room) for (long n1 : {0L, 1L, 5L, 22L}) for (long n2 : {0L, 1L, 9L, 40L}) {
        if (n1 + n2 == 0) continue;
        const double a = launch_rows(n1, 7.5, n2, 3.5, ncu, room), b = plain(n1, 7.5, n2, 3.5, ncu, room);
        ++cases;
        if (!(std::abs(a - b) <= 3.5 * (1.0 + kSharing * (room - 1)) + 1e-6)) { printf("model %d %d %ld %ld: %g %g\n", ncu, room, n1, n2, a, b); ++bad; }
    }
    printf("cases %ld bad %ld\n", cases, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                    reason="needs g++ and the HIP headers")
def test_default_tiling_covers_the_domain_and_model_agrees(tmp_path):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM_INCLUDE}", f"-I{CSRC}", str(src),
                    "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "bad 0" in r.stdout
