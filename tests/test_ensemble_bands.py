"""The row bands of an ensemble on the host (csrc/swe_tiling.h): a given height
is the height of every band; the chosen ones stay within their range, cover
every row of every member once and need no more items than one-row bands."""

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
#include <random>
using namespace swe;
using Shapes = std::vector<std::pair<int, int>>;

static long bad = 0, cases = 0;

static void check(const Shapes &shapes, int rows, int cus)
{
    const EnsBands b = ensemble_bands(shapes, rows, cus);
    ++cases;
    if (rows) { if (b.by != rows || b.tail != 0) { ++bad; printf("rows %d: by %d tail %d of %d\n", rows, b.by, b.tail, b.by2); } }
    else bad += b.by < 1 || b.by > 16 || b.tail < 0 || (b.tail > 0 && (b.by2 < 1 || b.by2 > 4 || b.by2 >= b.by));
    for (const auto &s : shapes) {
        const Tiling T = b.of(s.first, s.second);
        bad += (int64_t)T.ntiles > (int64_t)make_tiling(s.first, s.second, 1).ntiles;
        if (rows) bad += T.ntiles != make_tiling(s.first, s.second, rows).ntiles;
        std::vector<unsigned char> seen((size_t)T.nstrips * s.second, 0);
        for (int t = 0; t < T.ntiles; ++t) {
            int strip, y0, y1;
            tile_place(T, t, s.second, strip, y0, y1);
            if (strip < 0 || strip >= T.nstrips || y0 < 0 || y0 >= y1 || y1 > s.second) { ++bad; continue; }
            for (int y = y0; y < y1; ++y) seen[(size_t)strip * s.second + y]++;
        }
        for (unsigned char v : seen) bad += v != 1;
    }
}

int main()
{
    std::mt19937 r(3);
    std::vector<Shapes> sets = {{{2, 2}}, {{2600, 900}}, {{2600, 9000}}, {{2, 2}, {700, 333}, {64, 64}, {181, 600}, {1000, 3}},
                                {{61, 1}, {60, 2}, {59, 17}}};
    for (int n : {3, 12, 48, 256}) {
        Shapes s;
        for (int k = 0; k < n; ++k) s.push_back({200 + (int)(r() % 800), 200 + (int)(r() % 400)});
        sets.push_back(s);
    }
    for (const auto &s : sets)
        for (int cus : {256, 64})
            for (int rows : {0, 1, 2, 7, 16, 64, 4096}) check(s, rows, cus);
    printf("cases %ld bad %ld\n", cases, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                    reason="needs g++ and the HIP headers")
def test_ensemble_bands(tmp_path):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROCM_INCLUDE}", f"-I{CSRC}", str(src), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]


GRID = r"""
#include "swe_tiling.h"
#include <cstdio>
using namespace swe;
int main()
{
    long bad = 0;
    const int64_t items[] = {1, 4, 4096, 1 << 20, ((int64_t)1 << 26) - 64, (int64_t)1 << 26, ((int64_t)1 << 27) + 5, (int64_t)1 << 31};
    for (int64_t n : items) for (int chunk : {0, 1, 3, 64, 1024}) {
        const int c = ensemble_chunk(n, chunk);
        const int64_t blocks = ensemble_blocks(n, c);
        // every item has a wave, blocks come in eights, and a launch has fewer
        // than 2^32 threads
        if (c < 1 || blocks * kWavesPerBlock * c < n || blocks % 8 || blocks * kWavesPerBlock * kWave >= ((int64_t)1 << 32)) { ++bad; printf("%lld %d: %d %lld\n", (long long)n, chunk, c, (long long)blocks); }
        // what is asked for is kept where it can be
        if (n < ((int64_t)1 << 26) - 64 && c != (chunk ? chunk : 1)) ++bad;
    }
    printf("bad %ld\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                    reason="needs g++ and the HIP headers")
def test_ensemble_grid_stays_below_the_launch_limit(tmp_path):
    src = tmp_path / "grid.cpp"
    src.write_text(GRID)
    exe = str(tmp_path / "grid")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROCM_INCLUDE}", f"-I{CSRC}", str(src), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
