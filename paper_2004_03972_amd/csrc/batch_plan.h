// batch_plan.h -- tile shape, kernel and placement of the batched step (host code, plain C++).
//
// All figures are microseconds per step unless said otherwise.  The lines were drawn from 220
// random batches (1 to 100 instances of 100 to 8000 spins, 1 to 512 replicas, each storage form
// and mixtures), each timed in every shape, kernel and placement: against the best of those the
// rules cost 2% on average; 200 further batches took 0.73 of the time of one kernel for all, 64
// replicas, eight wavefronts and whole instances an XCD, and at worst 1.08 of it.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace hqa {

constexpr int BL_ROWS = 128;      // rows of a tile

struct BatchTile {
    int inst, i0, r0, pad;
};

struct BatchShape {
    int inst;        // index in the handle
    int N, Np;
    int form;        // streamed couplings: 0 FP32, 1 BF16, 2 FP8, 3 one bit
};

struct BatchForm {
    int rt;          // replica tiles of 16 per workgroup
    bool wide;       // four wavefronts of 32-row tiles (rt = 4)
    bool stream;     // ... and the state passes the last-level cache by
};

inline int64_t batch_row_tiles(int N) { return ((int64_t)N + BL_ROWS - 1) / BL_ROWS; }

// What a step reads and writes: the couplings, and per spin two copies of phi and of its BF16
// operand, p and S.
inline int64_t batch_coupling_bytes(const BatchShape &s) {
    const int64_t cells = (int64_t)s.Np * s.Np;
    return s.form == 0 ? 4 * cells : s.form == 1 ? 2 * cells : s.form == 2 ? cells : cells / 8;
}

inline int64_t batch_bytes(const std::vector<BatchShape> &inst, int R) {
    int64_t b = 0;
    for (const BatchShape &s : inst) b += batch_coupling_bytes(s) + 20ll * s.N * R;
    return b;
}

// The kernel of the BF16 and FP8 instances `inst`; bytes: of the whole handle.
//
// Tiles of 64 replicas are all resident at once up to 512 (two per CU).  Few of them leave a step
// waiting on its longest tile, whose groups run at the latency of one or two workgroups per CU,
//  * up to 16 replicas take 16 a tile, up to 32 take 32;
//  * up to 96 tiles of 64: 16 (R = 64, 64 / 32 / 16 replicas a tile: 88 tiles 30.5 / 18.8 / 16.3, 17
//    instances of 1280 spins, 170 tiles, 19.3 / 15.8 / 23.4; R = 31, 9 of 100 .. 4309 35.5 / 21.9 /
//    24.7);
//  * up to 560 tiles of 32 (one-bit couplings, of which halved tiles read little: 1280): 32, as long
//    as the couplings that are then read twice are near (150 MB; 64 / 32 replicas a tile: R = 100,
//    444 tiles of 32 13.1 / 11.9; R = 128, 496, 54 MB 19.9 / 17.5, 158 MB 41.8 / 47.5; 604 18.1 /
//    19.3; 698 30.2 / 32.9);
//  * R = 65 .. 96 takes three 32s rather than two 64s up to the last-level cache's 256 MB (R = 65,
//    990 tiles of 64 51.4 / 41.8).
// Beyond that cache the state passes it by, which leaves it to the couplings and operands (kept /
// passed by: 24 instances R = 64, 102 MB 40.6 / 42.2; N = 8192, R = 768, 190 MB 128 / 150; 265 MB
// 137.6 / 144.9; 271 MB 125 / 120; 60 instances, 294 MB 104 / 93; 100 instances, 464 MB 152 / 138;
// couplings passed by as well: 60 instances 141).  From 1400 MB on the cache holds little of the
// couplings either way, and where they are few beside the state (at most 0.4 of it, or one bit each
// in two tiles of three) eight wavefronts cover its reads better (state kept, eight wavefronts /
// passed by, four: one bit, 1115 of 1351 642 / 692, 265 of 3686 691 / 724; FP8, R = 256, 227 of
// 1376 559 / 601; 512 of the uneven batch 724 / 729; but BF16 310 of 1276 .. 1658 287 / 265).  66
// large batches are 0.1% off the better of the two in the mean, 2% at worst.
// Four wavefronts of 32-row tiles multiply faster, eight of 16-row tiles have the shorter way
// through a tile.  So four take batches of more than 512 tiles whose mean tile passes at least 2400
// columns (eight / four: 20 instances of 3792 267 / 257, 22 of 2827 120 / 115; 26 of 1632 164 / 163,
// 67 of 194 .. 667 42.7 / 46.7, 65 of 413 .. 616 47.9 / 52.9), and a single instance unless its BF16
// couplings pass few groups (N = 8192, R = 512, FP8 92 / 80, BF16 111 / 102; BF16 N = 2048, R = 2048
// 43 / 47).
inline BatchForm batch_form_for(const std::vector<BatchShape> &inst, int R, int64_t bytes) {
    int64_t rows = 0, cols = 0, bit_rows = 0, coupling = 0, state = 0;
    bool bits = true, few = false;
    for (const BatchShape &s : inst) {
        const int64_t n = batch_row_tiles(s.N);
        rows += n;
        cols += n * s.Np;
        if (s.form == 3) bit_rows += n;
        coupling += batch_coupling_bytes(s);
        state += 20ll * s.N * R;
        bits &= s.form == 3;
        few |= s.form == 1 && s.Np < 4096;
    }
    const int64_t c32 = rows * (((int64_t)R + 31) / 32), c64 = rows * (((int64_t)R + 63) / 64);
    const int64_t MB = (int64_t)1 << 20;
    BatchForm f = {4, false, false};
    if (R <= 16 || c64 <= 96) f.rt = 1;
    else if (R <= 32 || (c32 <= (bits ? 1280 : 560) && bytes <= 150 * MB) ||
             (R > 64 && R <= 96 && bytes <= 256 * MB)) f.rt = 2;
    if (f.rt == 4) {
        const bool light = inst.size() > 1 && bytes > 1400 * MB &&
                           (5 * coupling <= 2 * state || 3 * bit_rows >= 2 * rows);
        f.stream = bytes > 256 * MB && !light;
        f.wide = f.stream || (c64 > 512 && cols >= 2400 * rows && !light) || (inst.size() == 1 && !few);
    }
    return f;
}

constexpr int BATCH_XCDS = 8, BATCH_CUS = 32;   // XCDs, and compute units of each

// Tiles of each XCD, largest padded size first (`inst` comes in that order).  Each instance goes
// to the least-loaded XCD (longest processing time first), so that its flux operand is fetched
// into one L2; with `spread` each tile does.  An instance with at least an eighth of all the work
// is split in either case: its row blocks are cut into eight contiguous ranges, one per XCD, each
// with all replica tiles, so every XCD reads an eighth of J.
inline void batch_lists(const std::vector<BatchShape> &inst, int R, int reps, bool spread,
                        std::vector<BatchTile> (&xl)[BATCH_XCDS]) {
    int64_t load[BATCH_XCDS] = {0}, total = 0;
    const int64_t rts = ((int64_t)R + reps - 1) / reps;
    // work of a tile: the bytes it streams (its couplings and the staged flux block) plus a fixed
    // cost of its first loads and epilogue (about the time of 256 KB)
    auto tile_work = [&](const BatchShape &s) -> int64_t {
        const int64_t jb = s.form == 0 ? 512 : s.form == 1 ? 256 : s.form == 3 ? 16 : 128;
        return (jb + 2 * reps) * (int64_t)s.Np + 262144;
    };
    auto least = [&]() {
        int x = 0;
        for (int y = 1; y < BATCH_XCDS; y++)
            if (load[y] < load[x]) x = y;
        return x;
    };
    for (const BatchShape &s : inst) total += batch_row_tiles(s.N) * rts * tile_work(s);
    for (const BatchShape &s : inst) {
        const int nrb = (int)batch_row_tiles(s.N);
        const int64_t tw = tile_work(s), work = nrb * rts * tw;
        const bool split = nrb >= BATCH_XCDS && BATCH_XCDS * work >= total;
        const int whole = split || spread ? 0 : least();
        for (int rb = 0; rb < nrb; rb++)
            for (int r0 = 0; r0 < R; r0 += reps) {
                // split: row block rb lies in range x of the eight, x nrb / 8 <= rb
                const int x = split ? (int)((((int64_t)rb + 1) * BATCH_XCDS - 1) / nrb) : spread ? least() : whole;
                xl[x].push_back({s.inst, rb * BL_ROWS, r0, 0});
                load[x] += tw;
            }
    }
    // an XCD's first 32 tiles get a CU each, the others join them from the first CU on: longest
    // tiles last among the first, so that they are not joined by long ones (374 tiles: 44.0 -> 40.3)
    if (spread)
        for (auto &l : xl)
            if (l.size() > BATCH_CUS) std::reverse(l.begin(), l.begin() + BATCH_CUS);
}

// Estimate of a step: what the busiest CU of an XCD gets, 128-column groups and six more a tile
// for its prologue and epilogue, and `share` of what a CU of that XCD gets on average.
inline double batch_estimate(const std::vector<BatchTile> (&xl)[BATCH_XCDS], const std::vector<int> &groups,
                             double share) {
    double worst = 0.0;
    for (const auto &l : xl) {
        int64_t cu[BATCH_CUS] = {0}, sum = 0;
        for (size_t j = 0; j < l.size(); j++) {
            const int w = groups[l[j].inst] + 6;
            // two tiles a CU are resident from the start, later ones follow the first that ends
            int64_t *c = j < 2 * BATCH_CUS ? cu + j % BATCH_CUS : std::min_element(cu, cu + BATCH_CUS);
            *c += w;
            sum += w;
        }
        worst = std::max(worst, (double)*std::max_element(cu, cu + BATCH_CUS) + share * (double)sum / BATCH_CUS);
    }
    return worst;
}

// The launch order of a family's tiles (workgroup b runs on XCD b mod 8), padded with placeholders
// of instance -1.  Whole instances an XCD keep one L2 per operand, tiles one by one even out the
// XCDs but have the fluxes fetched into several L2s, and the couplings of a row block into one more
// for each further replica tile.  So tiles go one by one where that is estimated better by more
// than 3%, a group, and 0.15 of a group for each MB fetched again (instance by instance / tile by
// tile: 24 uneven instances, estimates 115 and 75, 55.4 / 40.3; 9 of 248 .. 4392, R = 69, 91 and 78,
// 28.0 / 25.6; 20 of 3414, R = 64, 539 MB 166.6 / 145.0; against: 34 of 148, R = 256 14.0 / 17.1, 58 of
// 101 .. 404, R = 100 16.0 / 17.9, 30 of 1062 .. 1593, R = 64 23.8 / 26.4, and 13 of 768 .. 2129 in BF16,
// R = 65, 96 MB of couplings fetched again, 38.8 / 43.8); in FP32, whose tiles compute longer, better
// by more than 5% (12 of 2268 .. 3293, R = 8 181 / 158; 24 of 185 .. 267, R = 200 22.4 / 24.1).  Beyond
// 1024 tiles of 64 replicas XCDs are even as they are (26 of 1632, R = 282, 1690 tiles 144 / 177).
inline std::vector<BatchTile> batch_place(const std::vector<BatchShape> &inst, int R, int reps, bool f32) {
    std::vector<BatchTile> xl[BATCH_XCDS], one[BATCH_XCDS], out;
    if (inst.empty()) return out;
    batch_lists(inst, R, reps, false, xl);
    const int64_t rts = ((int64_t)R + reps - 1) / reps;
    int64_t c64 = 0;
    double again = 0.0;                                // MB
    int last = 0;
    for (const BatchShape &s : inst) {
        const double cells = (double)s.Np * s.Np;
        c64 += batch_row_tiles(s.N) * (((int64_t)R + 63) / 64);
        again += 1e-6 * ((s.form == 1 ? 2.0 : s.form == 2 ? 1.0 : 0.125) * cells *
                             (double)(std::min<int64_t>(rts, BATCH_XCDS) - 1) +
                         2.0 * s.Np * R);
        last = std::max(last, s.inst);
    }
    if (c64 <= 1024) {
        std::vector<int> groups(last + 1, 0);
        for (const BatchShape &s : inst) groups[s.inst] = s.Np / 128;
        batch_lists(inst, R, reps, true, one);
        const double share = f32 ? 0.3 : 0.6;
        const double whole = batch_estimate(xl, groups, share), single = batch_estimate(one, groups, share);
        if (whole > (f32 ? 1.05 * single : 1.03 * single + 1.0 + 0.15 * again))
            for (int x = 0; x < BATCH_XCDS; x++) xl[x].swap(one[x]);
    }
    size_t longest = 0;
    for (const auto &l : xl) longest = std::max(longest, l.size());
    for (size_t j = 0; j < longest; j++)
        for (const auto &l : xl) out.push_back(j < l.size() ? l[j] : BatchTile{-1, 0, 0, 0});
    return out;
}

}  // namespace hqa
