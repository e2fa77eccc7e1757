// Host arithmetic of the launches, free of HIP so that it can be compiled and
// checked on its own: the cut of a packing's rows into work items, what runs an
// iteration's tail, how many iterations are launched in a row, and grids that
// grow with the number of packings.
#pragma once
#include "rcp.h"

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace rcp {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

// The cut of the rows into work items, one a wave, four a block (the kernels
// that take a block's rows together join its four): a row costs row_units
// plus one per partner, an item holds item_units.  A wave takes a sixth
// of the tuning's item_work, and a row two thirds of its row_cost: by the
// defaults (6, 1536) 256 units at 4 a row, so up to 64 rows, about 40 on the
// dense million-sphere state (2.3 partners a row).  Measured there, on 3e6
// spheres of size ratio 5e5 and on 1e5 spheres with 5.2 partners, us per
// launch: 42.2 / 126 / 13.8; with a quarter of both, 384 units at 6, 42.8 /
// 127 / 16.0, with 256 at 5 46.7 / 130 / 14.3, with 192 at 3 43.1 / 128 /
// 13.7 (and more partials for the tail).
//
// The wave kernels hold a row a lane, so their items have at most 64 rows:
// item_work <= 256 row_cost gives no more.  With variant bit 5 (512 row_cost)
// an item may have 128, for the kernel that takes 512 rows a block; `waves`
// cuts it to 64.
//
// A packing of fewer than kFineItems such items is cut finer, down to one
// round of 64 entries an item: a wave of its own is then free for every
// round.  512 spheres with 13.6 partners, us per launch: 6.8 against 7.9.
// The rule looks at the packing alone (a batch must give it the same bits as
// a context of its own), so the line lies where a census of 16 packings of
// 2e3 to 3.4e4 spheres does not slow down: 12.7 us with 96 items, 14.1 with
// 128, 15.7 with 512, although 8784 spheres alone would gain by 512 (7.2
// against 8.7).
constexpr int64_t kFineItems = 96;

inline int row_units(const rcp_tuning &t) { return (2 * t.row_cost + 2) / 3; }

// Units of an item at most, whatever the packing.
inline int item_units_max(const rcp_tuning &t, bool waves)
{
    const int64_t wk = std::max(1, t.item_work / 6);
    return (int)(waves ? std::min<int64_t>(wk, (int64_t)kWave * row_units(t)) : wk);
}

// Rows of an item at most: row i has the work coordinate row_units i + rp[i],
// and an item the rows of one stretch of item_units of it.
inline int item_rows_max(const rcp_tuning &t, bool waves)
{
    return (item_units_max(t, waves) + row_units(t) - 1) / row_units(t);
}

inline int item_units(const rcp_tuning &t, bool waves, int64_t n, int64_t entries)
{
    const int64_t fine = (row_units(t) * n + entries) / kFineItems;
    return (int)std::min<int64_t>(item_units_max(t, waves), std::max<int64_t>(fine, kWave));
}

// Item slots for n rows and that many entries: enough for all units, plus
// one, in whole blocks.
inline int64_t item_slots(const rcp_tuning &t, bool waves, int64_t n, int64_t entries)
{
    const int64_t k = (row_units(t) * n + entries) / item_units(t, waves, n, entries) + 2;
    return (k + kWavesPerBlock - 1) / kWavesPerBlock * kWavesPerBlock;
}

// Whether the gradient kernel runs the tail itself: only the block-per-item
// kernels have that form, not the wave kernels (`waves`: nothing else runs,
// whatever the tuning), the persistent one (bit 3) or the one of 512 rows a
// block (bit 5).
inline bool fuses_tail(const rcp_tuning &t, bool waves)
{
    return t.fused_tail && !waves && !(t.variant & (8 | 32));
}

// Where a running packing stands, for the launches ahead of it.
struct RunAhead {
    int64_t iters;               // its iteration count
    int64_t since_it, interval;  // that at the last list build, or where the
                                 // schedule began after it; and between the
                                 // last two in the schedule (0: not known)
    double max_disp2, disp_lim;  // displacement^2 since the build, and its limit
    int64_t to_limit, to_end;    // iterations before a limit, and in the schedule
};

// Iterations to launch before the host next looks at the records, from one
// packing's side (see launch_span); K: one graph.
inline int64_t iterations_ahead(const RunAhead &p, int64_t K)
{
    const int64_t since = std::max<int64_t>(0, p.iters - p.since_it);
    int64_t r = K;
    if (p.interval > 0) {
        r = p.interval - since;
    } else if (since > 0 && p.max_disp2 > 0.0 && p.disp_lim > 0.0) {
        const double d = std::sqrt(p.max_disp2);
        const double est = d < p.disp_lim ? (double)since * (p.disp_lim / d - 1.0) : 0.0;
        const int64_t cap = std::max<int64_t>(K, 2 * since);
        r = est < (double)cap ? (int64_t)est : cap;
    }
    return std::min({r, p.to_limit, p.to_end});
}

// Iterations of a schedule from `done` of rung `rung` on (no more than 2^62).
inline int64_t schedule_left(const int64_t *budget, int n_rungs, int rung, int64_t done)
{
    constexpr int64_t most = (int64_t)1 << 62;
    int64_t left = 0;
    for (int r = rung; r < n_rungs; ++r) left = budget[r] < most - left ? left + budget[r] : most;
    return std::max<int64_t>(0, left - done);
}

// Blocks of kBlock threads a launch takes along x (fewer than 2^32 threads);
// along y and z it takes 65535, so the packings of a census lie along x.
constexpr int64_t kGridBlocks = (((int64_t)1 << 32) - 1) / kBlock;

// Blocks per packing for a pass over nseg packings of up to nmax spheres: about
// 8192 in all.
inline int64_t blocks_per_packing(int64_t nseg, int64_t nmax)
{
    const int64_t most = std::max<int64_t>(1, 8192 / nseg);
    return std::max<int64_t>(1, std::min((nmax + kBlock - 1) / kBlock, most));
}

// Packings a launch takes with a block for each digit of `bits` bits.
inline int64_t packings_per_scan(int bits) { return kGridBlocks >> bits; }

}  // namespace rcp
