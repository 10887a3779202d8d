// csr_plan.h -- which kernels a sparse instance's size takes (host code, plain C++).
#pragma once
#include <stdint.h>

namespace hqa {

struct CsrPlan {
    int rows;          // > 0: k_step_csr_rows with so many gathers in flight; 0: k_step_csr
    int vec;           // k_step_csr: replicas a lane,
    uint32_t chunks;   // chunks of 64 vec replicas,
    bool sliced;       // and whether an XCD serves one chunk at a time
};

// Workgroups of k_step_csr.
inline uint64_t csr_wave_blocks(int N, const CsrPlan &p) {
    const uint64_t nrb = ((uint64_t)N + 3) / 4;
    if (p.sliced && p.chunks < 8) return 8 * ((nrb + 8 / p.chunks - 1) / (8 / p.chunks));
    return nrb * p.chunks;
}

// N rows, nnz couplings, max_deg in the longest row, Rp replicas (padded to a multiple of 4).  d =
// nnz / N is the mean degree; G(N, d) a random graph, us per step.  Over 1100 cases (lattices,
// random graphs of N 800 .. 60,000 and d 2 .. 40, R 1 .. 1500), each timed in six forms, the rule is
// 2% off the fastest in the mean.
//
// Few rows for their degree (N < 600 d, 900 d at up to four replicas, where G(10^4, 12) takes 6.4 /
// 6.8; below 6500 rows, 4000 past 64 replicas or where a row is one batch of gathers): a step lasts
// as long as its longest chain of gathers, and a wavefront a row, indices through scalar loads and
// 16 gathers at once, has the shortest (wavefront a row / rows side by side: G(2000, 12) R = 4, 64,
// 512: 3.8, 4.3, 8.4 / 5.3, 5.5, 8.9; G(10^4, 30) R = 4, 64: 7.8, 10.1 / 10.3, 11.0; G(3388, 5) R = 8,
// 64: 3.9, 4.3 / 4.9, 5.1; G(5180, 6) R = 8: 4.2 / 5.1; the 16^3 lattice R = 8: 3.9 / 3.6).
// More rows: there are wavefronts enough, and lanes without a replica and lines shared by two
// chunks cost what they are; rows side by side (four replicas a lane) waste neither.  (Wavefront a
// row / rows: the 100^3 lattice R = 4, 64, 260: 302, 466, 1908 / 19, 260, 1181; the 46^3 lattice
// R = 4, 64: 30, 34 / 4.0, 18.8; G(10^5, 12) R = 4, 68: 36, 125 / 11.5, 70.6; G(10^5, 30) R = 4, 16,
// 68, 260: 49, 55, 265, 541 / 25, 44, 153, 497.)  By replicas:
//  * up to 64, one a lane (G(10^4, 30) R = 64: 9.9, two or four a lane 14.4, 14.8); it stays for many
//    rows of d >= 20 and 36 replicas or more (G(10^5, 30) R = 48: 97 / 104; G(3 10^4, 30) R = 64: 26.3
//    / 27.6);
//  * d < 10: wide lanes, the step being state traffic (16^3, R = 128: 5.5 / 5.0 / 5.1; R = 1024:
//    23.0 / - / 16.7; G(3000, 5) R = 256: 8.2 / - / 7.0), for many rows in whole chunks of 256 only
//    (46^3, R = 256, 512: 104, 208 / 107, 213; 16^3, R = 512: 7.6 / 8.3);
//  * d >= 10 and chunks of 64 that fill the XCDs evenly and are nine tenths full: sliced over the XCDs,
//    many rows or few (G(10^4, 30) R = 256: 24.3, unsliced 35.0, four a lane 34.6; R = 128: 14.6, 16.0,
//    two a lane 16.2; G(10^5, 30) R = 128, 256, 1024: 214, 423, 1712 / rows 230, 469, 1868; G(13186, 12)
//    R = 1000: 92 / 113; two chunks for 80 replicas of G(20287, 40) 39.5 / 25.4);
//  * d >= 20 and 6.4 MB of fluxes or more (an XCD's L2 has 4): rows, two gathers in flight, with more
//    of them a line is lost before it is read again (G(10^5, 30) R = 68, 192: 153, 332, six 159, 344; G(7329, 30) R = 768:
//    70.5, six 88.9, a wavefront a row 91.7; G(9978, 40) R = 300: 48.7, 56.4, 61.7; below: G(7278, 30)
//    R = 100: 14.9, 11.8, 11.3);
//  * else rows for many, for few one or four replicas a lane (G(8386, 18) R = 160: 15.0 / 12.6).
// Six gathers in flight were best or within 3% of it in 16 graphs otherwise.
inline CsrPlan csr_plan(int N, int64_t nnz, int max_deg, uint32_t Rp) {
    const uint32_t nc = (Rp + 63) / 64;
    const bool d10 = nnz >= 10 * (int64_t)N, d20 = nnz >= 20 * (int64_t)N;
    const bool many = (double)N * N >= (Rp > 4 ? 600.0 : 900.0) * (double)nnz &&
                      N >= (Rp > 64 || max_deg <= 6 ? 4000 : 6500);
    const bool sliced = (nc == 2 || nc == 4 || nc % 8 == 0) && 10 * (uint64_t)Rp >= 9 * 64 * (uint64_t)nc;
    const CsrPlan rows = {6, 0, 0, false};
    CsrPlan p = {0, 1, nc, false};
    if (nc == 1) {
        if (many && !(d20 && Rp > 32)) return rows;
    } else if (!d10) {
        if (many && Rp % 256 != 0) return rows;
        p.vec = Rp <= 128 ? 2 : 4;
    } else if (sliced) {
        p.sliced = true;
    } else if (d20 && (uint64_t)N * Rp >= 1600000) {
        return {2, 0, 0, false};
    } else if (many) {
        return rows;
    } else if (nc > 2) {
        p.vec = 4;
    }
    p.chunks = (Rp + 64 * p.vec - 1) / (64 * p.vec);
    // a launch has fewer than 2^32 threads; rows side by side are N Rp / 4 of them
    return csr_wave_blocks(N, p) * 256 < ((uint64_t)1 << 32) ? p : rows;
}

// Whether the grids of the kernels that turn a replica-minor state in LDS (tiles of 32 spins x 32
// replicas in k_export_turn, 16 x 32 in k_features_turn) stay within 2^32 threads and 65,535 blocks
// in the second dimension; larger states take the kernels that do not.
inline bool export_turn_fits(int N) { return ((uint64_t)N + 31) / 32 * 256 < ((uint64_t)1 << 32); }
inline bool features_turn_fits(int N, int R) {
    return ((uint64_t)N + 15) / 16 * 512 < ((uint64_t)1 << 32) && ((int64_t)R + 31) / 32 <= 65535;
}

}  // namespace hqa
