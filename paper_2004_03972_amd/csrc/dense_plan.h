// dense_plan.h -- form of the dense per-step kernel by size: block shape where it was neither tuned
// nor pinned, and the tiled form's copies (host code, plain C++).
#pragma once
#include <stdint.h>

namespace hqa {

struct StepBlock {
    int tm, tn;      // a workgroup's output tiles of 16 rows x 16 replicas
    int cb;          // chunks of each chain's loads in flight together
};

inline int64_t step_blocks(int Np, int Rp, int tm, int tn) {
    return (int64_t)(Np / (16 * tm)) * (Rp / (16 * tn));
}

// Np rows (a multiple of 128), Rp replicas (a multiple of 16).
//
// Shape: workgroups come in turns of 256, one a CU, and a workgroup of 2 x 4, 2 x 2, 2 x 1 tiles
// lasts about 3.8, 2.2, 1.5 times as long as one of 1 x 1; the least sum of turns wins, the larger
// shape at equal sums.  Over 240 random sizes (N 60 ... 9000, R 1 ... 1500, three storage types) it
// is within 0.5% of the fastest of six shapes and two depths in the mean; the largest shape that
// gives 180 workgroups is 4.5% off, since a chip filled by 130 ... 180 large blocks beats two turns
// of smaller ones (us per step, this / 180: BF16 N = 5445, R = 13: 18.3 / 22.9; binary32 N = 4469,
// R = 19: 36.3 / 55.4; N = 5035, R = 60: 65.5 / 99.3; FP8 N = 1415, R = 44: 7.7 / 9.1).
//
// Depth: four chunks keep a chip with one workgroup a CU busy, and eight of 16- or 8-bit operands
// cost it up to a fifth (FP8 N = 3242, R = 637: 95.9 / 112.7; N = 7269, R = 436: 274 / 300).
// Binary32 operands, twice the bytes a product, gain from eight once a CU has two workgroups, and
// lose with fewer, which stand idle for longer before their first products (four / eight at
// N = 4461, R = 229: 259 / 219; N = 3556, R = 609: 405 / 342; N = 8756, R = 384: 628 / 496; with 160
// workgroups, N = 5035, R = 60: 65.5 / 76.5) -- and where a chain has two batches of eight, 1024
// columns (N = 332, R = 763: 11.3 / 12.9; N = 131, R = 1295: 9.0 / 11.0; N = 1044, R = 974: 68.5 / 62.8).
inline StepBlock step_block(int Np, int Rp, bool f32) {
    static const struct { int tm, tn; double w; } shapes[] = {
        {2, 4, 3.8}, {2, 2, 2.2}, {2, 1, 1.5}, {1, 1, 1.0}};
    StepBlock best = {1, 1, 4};
    double cost = 0;
    for (const auto &s : shapes) {
        if (Rp % (16 * s.tn)) continue;
        const double c = s.w * (double)((step_blocks(Np, Rp, s.tm, s.tn) + 255) / 256);
        if (cost != 0 && c >= cost) continue;
        cost = c;
        best.tm = s.tm;
        best.tn = s.tn;
    }
    if (f32 && Np >= 1024 && best.tm == 2 && step_blocks(Np, Rp, best.tm, best.tn) >= 512) best.cb = 8;
    return best;
}

// Whether a run of some steps by the tiled form reads the operand-order copies.  Setting the fluxes'
// copy up is a launch more on each run, some 2.4 us, and a step gains about 0.9 us per 1000 columns
// by it; shorter runs read the row-major state and couplings, bit for bit the same (us per step of
// runs of one step, tiled / row-major: N = 387 6.2 / 4.4, N = 1000 6.6 / 5.3, N = 2048 7.5 / 6.9,
// N = 4000 9.7 / 10.2; of two: N = 1000 5.5 / 5.3, N = 1500 6.0 / 6.1; of four: N = 387 4.4 / 4.4,
// N = 1000 4.9 / 5.2).
inline bool step_reads_tiles(int Np, int64_t steps) { return steps >= 2560 || steps * Np >= 2560; }

}  // namespace hqa
