"""A block at the top of the arena (csrc/swe_arena.h: alloc_top), given back as
soon as another allocation needs the room, leaves every other allocation where
it lies without that block: random sequences against an arena that never has
one."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1912_02457_amd", "csrc")

CHECK = r"""
#include "swe_arena.h"
#include <cstdio>
#include <random>
#include <vector>
using namespace swe;
int main()
{
    long bad = 0, tops = 0, given = 0, refused = 0;
    std::mt19937 r(5);
    for (int run = 0; run < 400; ++run) {
        const size_t size = 256 * (20 + r() % 200);
        Arena a, b;  // with and without a block at the top
        a.reset(size);
        b.reset(size);
        size_t top = 0, top_bytes = 0;
        std::vector<std::pair<size_t, size_t>> live;
        for (int k = 0; k < 300; ++k) {
            const int what = r() % 8;
            if (what < 4) {
                const size_t n = 1 + r() % (256 * 30);
                size_t oa = 0, ob = 0;
                const bool gb = b.alloc(n, &ob);
                bool ga = a.alloc(n, &oa);
                if (!ga && top_bytes) {
                    Arena t = a;
                    t.release(top, top_bytes);
                    if (t.alloc(n, &oa)) { a.release(top, top_bytes); top_bytes = 0; ++given; ga = a.alloc(n, &oa); }
                }
                bad += ga != gb || (ga && oa != ob);
                refused += !gb;
                if (gb) live.push_back({ob, n});
            } else if (what < 6 && !live.empty()) {
                const size_t q = r() % live.size();
                a.release(live[q].first, live[q].second);
                b.release(live[q].first, live[q].second);
                live[q] = live.back();
                live.pop_back();
            } else if (what == 6 && !top_bytes) {
                const size_t n = 1 + r() % (256 * 40);
                if (a.alloc_top(n, &top)) {
                    top_bytes = n;
                    ++tops;
                    bad += top % kArenaAlign != 0 || top + n > size;
                    for (auto &l : live) bad += l.first < top + n && top < l.first + l.second;
                }
            } else if (what == 7 && top_bytes) {
                a.release(top, top_bytes);
                top_bytes = 0;
            }
            bad += a.used() != b.used() + (top_bytes ? arena_align_up(top_bytes) : 0);
        }
    }
    printf("tops %ld given back %ld refused %ld bad %ld\n", tops, given, refused, bad);
    return bad != 0 || tops < 100 || given < 20 || refused < 100;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_top_block_leaves_the_others_in_place(tmp_path):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", f"-I{CSRC}", str(src), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout + r.stderr[-2000:]
