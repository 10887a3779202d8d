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

// N rows, nnz couplings, Rp replicas (padded to a multiple of 4).  d = nnz / N is the mean degree.
//
// Few rows for their degree (N < 600 d, 900 d at up to four replicas, where G(10^4, 12) takes 6.4 /
// 6.8): a step lasts as long as its longest chain of gathers, and a wavefront a row, indices
// through scalar loads and 16 gathers at once, has the shortest (us per step, wavefront a row / rows side by side: G(2000, 12) R = 4, 64, 512: 3.8, 4.3, 8.4 / 5.3, 5.5,
// 8.9; G(10^4, 30) R = 4, 64: 7.8, 10.1 / 10.3, 11.0; the 8^3 lattice R = 4: 3.7 / 3.4).  It takes
//  * up to 64 replicas: one a lane (G(10^4, 30) R = 64: 9.9, two or four a lane 14.4, 14.8);
//  * d < 10: wide lanes, the step being state traffic (16^3, R = 128: 5.5 / 5.0 / 5.1; R = 1024:
//    23.0 / - / 16.7; G(3000, 5) R = 256: 8.2 / - / 7.0);
//  * else 64-replica chunks, sliced over the XCDs when the chunks fill them evenly (G(10^4, 30)
//    R = 256: 24.3, unsliced 35.0, four a lane 34.6; R = 128: 14.6, 16.0, two a lane 16.2); an
//    uneven number of chunks above three takes four a lane.
// More rows: there are wavefronts enough, and lanes without a replica and lines shared by two
// chunks cost what they are; rows side by side (four replicas a lane) waste neither.  (Wavefront a
// row / rows: the 100^3 lattice R = 4, 64, 260: 302, 466, 1908 / 19, 260, 1181; the 46^3 lattice
// R = 4, 64: 30, 34 / 4.0, 18.8; G(10^5, 12) R = 4, 68: 36, 125 / 11.5, 70.6; G(10^5, 30) R = 4, 16,
// 68, 260: 49, 55, 265, 541 / 25, 44, 153, 497.)  A wavefront a row stays for
//  * d < 10 and whole chunks of 256 (46^3, R = 256, 512: 104, 208 / 107, 213; 16^3, R = 512: 7.6 /
//    8.3);
//  * d >= 10 and whole chunks that fill the XCDs evenly (G(10^5, 30) R = 128, 256, 1024: 214, 423,
//    1712 / 230, 469, 1868; G(3 10^4, 30): 48, 92, 356 / 59, 131, 564);
//  * d >= 20 and 36 to 64 replicas (G(10^5, 30) R = 48: 97 / 104; G(3 10^4, 30) R = 64: 26.3 / 27.6).
// Six gathers in flight were best or within 3% of it in 16 graphs; long rows of more than 64
// replicas (d >= 20) take two, with more of them the L2 loses lines before they are read again
// (G(10^5, 30) R = 68, 192: 153, 332, six 159, 344).
inline CsrPlan csr_plan(int N, int64_t nnz, uint32_t Rp) {
    const uint32_t nc = (Rp + 63) / 64;
    const bool even = nc == 2 || nc == 4 || nc % 8 == 0;
    const bool d10 = nnz >= 10 * (int64_t)N, d20 = nnz >= 20 * (int64_t)N;
    const CsrPlan rows = {d20 && Rp > 64 ? 2 : 6, 0, 0, false};
    if ((double)N * N >= (Rp > 4 ? 600.0 : 900.0) * (double)nnz) {
        const bool wave = !d10 ? Rp % 256 == 0 : Rp > 64 ? even && Rp % 64 == 0 : d20 && Rp > 32;
        if (!wave) return rows;
    }
    CsrPlan p = {0, 1, nc, false};
    if (nc > 1) {
        if (!d10) p.vec = Rp <= 128 ? 2 : 4;
        else if (even) p.sliced = true;
        else if (nc != 3) p.vec = 4;
        p.chunks = (Rp + 64 * p.vec - 1) / (64 * p.vec);
    }
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
