"""The pool of staging buffers (csrc/swe_staging.h) on the host: a call never
waits for another's buffer and never shares one, what is idle is reused, what
is kept stays within its bounds, and trimming leaves one buffer."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1912_02457_amd", "csrc")

CHECK = r"""
#include "swe_staging.h"
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <thread>
#include <vector>
using namespace swe;

static std::mutex mu;
static std::map<char *, size_t> held;  // everything got and not put back
static std::atomic<long> gets{0};
static std::atomic<bool> none{false};
struct Fake {  // addresses only: nothing the size of a real buffer is touched
    static char *get(size_t n)
    {
        if (none) return nullptr;
        ++gets;
        char *p = (char *)std::malloc(64);
        std::lock_guard<std::mutex> lk(mu);
        held[p] = n;
        return p;
    }
    static void put(char *p)
    {
        { std::lock_guard<std::mutex> lk(mu); if (!held.erase(p)) std::abort(); }
        std::free(p);
    }
};
static size_t total() { std::lock_guard<std::mutex> lk(mu); size_t t = 0; for (auto &h : held) t += h.second; return t; }
static long bad = 0;
#define CHECK(c) do { if (!(c)) { ++bad; std::printf("FAIL line %d: %s\n", __LINE__, #c); } } while (0)

int main()
{
    const size_t MiB = (size_t)1 << 20;
    {   // one after the other: one buffer serves every smaller call
        StagePool<Fake> p;
        for (int k = 0; k < 100; ++k) { StageBuffer b = p.take(8 * MiB); CHECK(b.p && b.bytes >= 8 * MiB); p.give(b); b = p.take(k * 1000 + 1); p.give(b); }
        CHECK(gets == 1 && held.size() == 1);
        p.trim();
        CHECK(held.size() == 1);
        Fake::put(held.begin()->first);
    }
    {   // side by side: a buffer each, none shared
        StagePool<Fake> p;
        std::vector<StageBuffer> v;
        for (int k = 0; k < 40; ++k) v.push_back(p.take(MiB));
        for (int k = 0; k < 40; ++k) for (int q = 0; q < k; ++q) CHECK(v[k].p != v[q].p);
        for (auto &b : v) p.give(b);
        CHECK(held.size() <= (size_t)kStageSlots && total() <= kStageKept);
        p.trim();
        CHECK(held.size() == 1);
        // small ones make room for large ones, beyond the bound nothing is kept
        for (int k = 0; k < 10; ++k) { StageBuffer a = p.take(kStageCap), b = p.take(kStageCap), c = p.take(kStageCap); p.give(a); p.give(b); p.give(c); }
        CHECK(total() <= kStageKept);
        const long g = gets;
        StageBuffer a = p.take(kStageCap);
        CHECK(gets == g);
        p.give(a);
        a = p.take(kStageKept + 1);
        CHECK(a.p && a.bytes > kStageKept);
        p.give(a);
        CHECK(total() <= kStageKept && total() >= 3 * kStageCap);
        none = true;
        a = p.take(kStageKept + 1);
        CHECK(!a.p && a.bytes == 0);
        p.give(a);
        none = false;
        p.trim();
        Fake::put(held.begin()->first);
        CHECK(held.empty());
    }
    {   // ever larger calls pin memory a few times, and little more than they need
        StagePool<Fake> p;
        const long g = gets;
        for (size_t n = 100 * 1000; n <= kStageCap; n += 500 * 1000) {
            StageBuffer b = p.take(n);
            CHECK(b.p && b.bytes >= n && b.bytes <= std::max(2 * n, (size_t)2 * MiB));
            p.give(b);
        }
        CHECK(gets - g <= 8 && total() <= kStageKept);
        p.trim();
        CHECK(held.size() == 1);
        Fake::put(held.begin()->first);
    }
    {   // threads: every buffer is one thread's at a time
        StagePool<Fake> p;
        std::vector<std::thread> ts;
        std::atomic<long> wrong{0};
        for (int t = 0; t < 8; ++t) ts.emplace_back([&, t] {
            for (int k = 0; k < 3000; ++k) {
                StageBuffer b = p.take((size_t)(1 + (k * 7 + t) % 40) * MiB);
                std::memset(b.p, t, 64);
                std::this_thread::yield();
                for (int q = 0; q < 64; ++q) wrong += b.p[q] != t;
                p.give(b);
            }
        });
        for (auto &t : ts) t.join();
        CHECK(wrong == 0 && total() <= kStageKept && held.size() <= (size_t)kStageSlots);
        p.trim();
        CHECK(held.size() == 1);
        Fake::put(held.begin()->first);
    }
    std::printf("bad %ld\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("san", ["address,undefined", "thread"])
def test_staging_pool(tmp_path, san):
    src = tmp_path / "check.cpp"
    src.write_text(CHECK)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", f"-fsanitize={san}", f"-I{CSRC}", str(src), "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
