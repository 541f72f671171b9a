// Host-side choice of a stage launch's tiling: the band heights (one, or a
// head and a tail of shorter bands) whose launch a small model of the chip
// finishes first.
//
// A launch is a queue of blocks of four waves, one per SIMD of a CU.  A band
// of `by` rows costs its rows and about kBandStart more (the halo rows it
// loads and reconstructs, the launch and the first loads).  The m blocks that
// share a CU get through c(m) = m / (1 + kSharing (m - 1)) rows at a time:
// one wave alone is a chain of dependent instructions, four keep the SIMD's
// issue busy.  What decides between tilings is how the blocks fill the CUs:
// 2.25 blocks per CU are as slow as three, and a tail of short bands evens out
// what the tall ones leave.
//
// The two constants and kOneHeight were fitted to event times of both stages,
// both state kinds, about 50 tilings of each of 15 domains from 128 x 128 to
// 4096 x 4096 (100 x 4000 and 4000 x 100 among them).  With the present kernels
// a launch at the tiling chosen takes on average 3 % longer than at the best
// one measured for it, at worst 15 % (2048 x 2048, stage 1); with gridded wind
// and the literal projection, which were not in the fit, 2 and 3 % and 9 %.
// A step in us with the rule before it (work spread over the wave slots plus
// one wave's chain, one band height, strip-major tiles) and with this one: 128
// x 128 13.3 and 9.1, 512 x 512 18.9 and 14.2, 1024 x 1024 beach 45 and 38,
// 2600 x 900 coast 72 and 57 (float32 state 63 and 50), 2048 x 2048 130 and
// 91, 4096 x 4096 590 and 420.
#pragma once

#include <algorithm>
#include <cmath>

#include "swe_device.h"

namespace swe {

constexpr int kMaxResident = 8;       // blocks per CU the model follows
constexpr double kBandStart = 1.5;    // rows
constexpr double kSharing = 0.4;
constexpr double kOneHeight = 1.1;    // bands of one height end less evenly than the model's

// CUs in the same state: `count` of them, each with n blocks, w[] rows left in each
struct CuGroup {
    int count, n;
    double w[kMaxResident], since;
};

// Time (in rows of one wave) until the last of n1 blocks of c1 rows and then
// n2 blocks of c2 rows is done, on ncu CUs with room for `room` blocks each.
// A group of CUs is split where one of the two queues runs out among its CUs,
// so there are never more than three (and no memory is allocated: this runs
// inside calls that have no way to report that there is none).
inline double launch_rows(long n1, double c1, long n2, double c2, int ncu, int room)
{
    // all but the last eight rounds of tall blocks run in step
    const long round = (long)ncu * room, extra = std::max(0L, n1 / round - 8);
    n1 -= extra * round;
    const double ahead = (double)extra * c1 * (1.0 + kSharing * (room - 1));
    CuGroup g[3] = {CuGroup{ncu, 0, {}, 0.0}};
    int ng = 1;
    // one more block for each CU of group k, split where the queue changes
    auto give = [&](int k) {
        while (n1 + n2 > 0) {
            long &left = n1 > 0 ? n1 : n2;
            const double c = n1 > 0 ? c1 : c2;
            if (left >= g[k].count) {
                left -= g[k].count;
                g[k].w[g[k].n++] = c;
                return;
            }
            CuGroup part = g[k];
            part.count = (int)left;
            part.w[part.n++] = c;
            g[k].count -= part.count;
            left = 0;
            g[ng++] = part;
        }
    };
    auto pace = [](int n) { return 1.0 / (1.0 + kSharing * (n - 1)); };  // rows per unit of time of each block
    for (int layer = 0; layer < room; ++layer)
        for (int k = 0, m = ng; k < m; ++k)
            if (g[k].n == layer) give(k);
    double last = 0.0;
    while (true) {
        int k = ng;
        double t = INFINITY;
        for (int q = 0; q < ng; ++q)
            if (g[q].n > 0) {
                const double e = g[q].since + *std::min_element(g[q].w, g[q].w + g[q].n) / pace(g[q].n);
                if (e < t) { t = e; k = q; }
            }
        if (k == ng) return ahead + last;
        last = t;
        CuGroup &x = g[k];
        const double done = (t - x.since) * pace(x.n);
        int n = 0;
        for (int q = 0; q < x.n; ++q)
            if (x.w[q] - done > 1e-9) x.w[n++] = x.w[q] - done;
        const int freed = x.n - n;
        x.n = n;
        x.since = t;
        const int before = ng;
        for (int q = 0; q < freed && n1 + n2 > 0; ++q) {
            give(k);
            // a part split off still waits for its other blocks
            for (int p = before; p < ng; ++p)
                for (int r = g[p].n - n; r < freed && n1 + n2 > 0 && r <= q; ++r) give(p);
        }
    }
}

// No launch of these blocks ends before this: the chip full until the end.
inline double launch_rows_least(long n1, double c1, long n2, double c2, int ncu, int room)
{
    return ((double)n1 * c1 + (double)n2 * c2) * (1.0 + kSharing * (room - 1)) / ((double)ncu * room);
}

// The tiling of one stage kernel on a chip of `cus` CUs where its registers
// allow `waves_per_simd` waves.
inline Tiling default_tiling(int nx, int ny, int cus, int waves_per_simd)
{
    // taller bands save a few more halo rows and lose more in the caches: 4096
    // x 4096 takes 413 us a step with the best tail to 16-row bands, 421 with
    // 24, 427 with 32 (float32 state 289, 288, 289)
    static const int heights[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16};
    const int room = std::min(std::max(waves_per_simd, 1), kMaxResident);
    const int nstrips = (nx + kStrip - 1) / kStrip;
    Tiling best = make_tiling(nx, ny, 1);
    double best_t = INFINITY;
    auto consider = [&](const Tiling &T) {
        const long n1 = T.nblk1, n2 = T.nblocks - T.nblk1;
        const double c1 = T.by + kBandStart, c2 = T.by2 + kBandStart;
        const double uneven = T.nrb1 == T.nrb && T.by > 1 ? kOneHeight : 1.0;
        if (launch_rows_least(n1, c1, n2, c2, cus, room) * uneven >= best_t) return;
        const double t = launch_rows(n1, c1, n2, c2, cus, room) * uneven;
        if (t < best_t) { best_t = t; best = T; }
    };
    for (int by : heights) {
        if (by > ny) break;
        consider(make_tiling(nx, ny, by));
        // tails of a quarter to two rounds of the wave slots
        for (int by2 = 1; by2 <= 4 && by2 < by; ++by2)
            for (double rounds : {0.25, 0.5, 1.0, 2.0}) {
                const int bands = std::max(1, (int)std::lround(rounds * cus * kWavesPerBlock * room / nstrips));
                if ((long)bands * by2 + by <= ny) consider(make_tiling_tail(nx, ny, by, by2, bands * by2));
            }
    }
    return best;
}

// Both stages' tilings: chosen once where the same number of waves of both fit
// (creating a 2600 x 900 domain takes 3600 us, a choice 60 of them).
inline void default_tilings(int nx, int ny, int cus, const int *waves_per_simd, Tiling *out)
{
    out[0] = default_tiling(nx, ny, cus, waves_per_simd[0]);
    out[1] = waves_per_simd[1] == waves_per_simd[0] ? out[0] : default_tiling(nx, ny, cus, waves_per_simd[1]);
}

// The bands of an ensemble's members: `by` rows, and after them, where tail is
// not 0, bands of by2 rows: at least `tail` of them in each member, and the
// rows that whole bands of `by` leave before those.  A member too short for
// both has one height.
struct EnsBands {
    int by, by2, tail;
    Tiling of(int nx, int ny) const { return make_tiling_tail(nx, ny, by, by2, by2 * tail < ny ? by2 * tail : 0); }
};

constexpr double kEnsembleStart = 1.0;  // rows more than kBandStart: the item and its member's fields
constexpr int kEnsembleRows = 16;       // where the workspace holds no more items than these bands give

// rows_per_wave > 0 is the height of every band; with 0 the same model as
// above chooses, over all members at once.
template <class Shapes>  // of (nx, ny) pairs
EnsBands ensemble_bands(const Shapes &shapes, int rows_per_wave, int cus)
{
    if (rows_per_wave) return EnsBands{rows_per_wave, 0, 0};
    static const int heights[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16};
    const int room = 4, nh = sizeof(heights) / sizeof(heights[0]);
    int64_t strips = 0, rows = 0;
    for (const auto &s : shapes) {
        const int64_t n = (s.first + kStrip - 1) / kStrip;
        strips += n;
        rows += n * s.second;
    }
    const int64_t slots = (int64_t)cus * kWavesPerBlock * room;
    EnsBands best{kEnsembleRows, 0, 0};
    const double per_slot = (double)rows / slots;
    double best_t = INFINITY;
    auto consider = [&](const EnsBands &b) {
        int64_t n1 = 0, n2 = 0;
        for (const auto &s : shapes) {
            const Tiling T = b.of(s.first, s.second);
            n1 += T.ntiles1;
            n2 += T.ntiles - T.ntiles1;
        }
        const double c1 = b.by + kBandStart + kEnsembleStart, c2 = b.by2 + kBandStart + kEnsembleStart;
        const double uneven = n2 == 0 && b.by > 1 ? kOneHeight : 1.0;
        n1 = (n1 + kWavesPerBlock - 1) / kWavesPerBlock;
        n2 = (n2 + kWavesPerBlock - 1) / kWavesPerBlock;
        if (launch_rows_least(n1, c1, n2, c2, cus, room) * uneven >= best_t) return;
        const double t = launch_rows(n1, c1, n2, c2, cus, room) * uneven;
        if (t < best_t) { best_t = t; best = b; }
    };
    for (int k = 0; k < nh; ++k) {
        const int h = heights[k];
        // the best bands hold 0.4 to 3 times a wave slot's share of the rows
        if (k < nh - 1 && (h > 3.0 * per_slot + 1.0 || h < 0.4 * per_slot - 1.0)) continue;
        if (k == nh - 1 && best_t < INFINITY && h > 3.0 * per_slot + 1.0) continue;
        consider(EnsBands{h, 0, 0});
        for (int by2 = 1; by2 <= 4 && by2 < h; ++by2)
            for (double rounds : {0.25, 0.5, 1.0}) {
                const int bands = (int)std::lround(rounds * slots / strips);
                if (bands > 0) consider(EnsBands{h, by2, bands});
            }
    }
    return best;
}

// Items per wavefront and blocks of an ensemble launch: `chunk` items (0: one)
// -- band heights already set how long a wave runs, and several items to a wave
// leave the last waves with uneven loads -- or as many more as keep a launch
// below 2^32 threads, the limit of a grid.
inline int ensemble_chunk(int64_t items, int chunk)
{
    const int64_t waves = ((((int64_t)1 << 32) / (kWavesPerBlock * kWave)) - 16) * kWavesPerBlock;
    return (int)std::max<int64_t>(chunk ? chunk : 1, (items + waves - 1) / waves);
}
// blocks of four waves, a multiple of the eight XCDs
inline int64_t ensemble_blocks(int64_t items, int chunk)
{
    const int64_t per_block = (int64_t)kWavesPerBlock * chunk;
    return ((items + per_block - 1) / per_block + 7) / 8 * 8;
}

}  // namespace swe
