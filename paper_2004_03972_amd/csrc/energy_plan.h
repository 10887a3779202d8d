// energy_plan.h -- launch shape and scratch of the exact energies (host code, plain C++).
//
// Dense instances run one launch of int8 digit products over all vectors (k_energy_mv in
// k_readout.hip): P slices of the couplings, each leaving a 64-bit word per digit for every vector
// and for the couplings' own sum, P D (V + 1) words.  Where the scratch does not hold those, the
// vectors go in several launches.
#pragma once
#include <stddef.h>

#include <algorithm>

namespace hqa {

// Digit counts the many-vector kernel is built for.
constexpr int MV_DIGITS[] = {1, 2, 4, 7, 8, 10, 12, 16, 20};
constexpr int MV_NDIGITS = 9;
constexpr size_t ACC_BYTES = 64;             // sizeof(Acc256)

// Slices of k_energy (one workgroup per vector and slice).
inline int energy_slices(int N, int V) {
    if (V <= 0) return 1;
    const int want = (512 + V - 1) / V;      // at least 512 workgroups in all
    const int most = (N + 63) / 64;          // at least 64 rows per slice
    return std::max(1, std::min(want, most));
}

// Bytes of scratch the energies of V vectors get, whatever the couplings.  It counts towards the
// fixed scratch of hqa_classify_noalloc, whose limit callers meet as HQA_EUNSUPPORTED, so it
// does not follow the launch: room for the partial sums of up to 1024 workgroups, and N bits a vector.
inline size_t energy_part_bytes(int N, int V) {
    V = std::max(V, 1);
    size_t m = 0;
    for (int L = 1; L <= 4; L++) {
        const int G = L == 1 ? 64 : L == 2 ? 32 : 16, groups = (V + G - 1) / G;
        const size_t P = std::max(1, std::min((1024 + groups - 1) / groups, (N + 15) / 16));
        m = std::max(m, 2 * P * L * ((size_t)V + 1));
    }
    const size_t by_vector = (size_t)V * energy_slices(N, V) * 2 * ACC_BYTES;
    return std::max(by_vector, (size_t)((V + 63) / 64) * N * 8 + m * 8 + 256);
}

// Vectors of a wavefront: up to 64 while the 4 D accumulators per 16 of them fit the registers.
inline int energy_mv_vec(int V, int D) { return V <= 16 || D > 12 ? 16 : D > 8 ? 32 : 64; }

// Whether k_energy scores V vectors of N spins sooner than digit products do.  At 16 spins a vector
// is one term a thread, and the products' merge, a digit at a time, is what a call waits for (us per
// call, digits / k_energy, N = 8: V = 100, 500, 2000, 8000 with D = 20 98, 105, 113, 137 / 71, 74, 89,
// 148; D = 10 82, 88, 95, 106 / 71, 73, 89, 150; D = 1 72, 78, 86, 93 / 62, 62, 65, 77; N = 16 and V =
// 2000 112, 92, 84 / 93, 92, 66; N = 32 and V = 2000 92, 92, 86 / 104, 104, 68).
inline bool energy_by_vector(int N, int V) { return N <= 16 && V <= 2048; }

struct EnergyPlan {
    int vec;      // vectors of a wavefront
    int P;        // slices
    int piece;    // vectors of a launch
};

// Slices: one or two workgroups per CU over the vector blocks (64-vector blocks fill the registers
// of one), each slice at least a block row.  Vectors of a launch: all, unless their sums would not
// fit in one slice (many vectors of few spins with wide spans: N = 100, V = 8192 at D = 20 takes
// two launches) or the grid's second dimension ends (65,535 blocks of vectors).
inline EnergyPlan energy_plan(int N, int V, int D) {
    EnergyPlan p;
    const size_t words = energy_part_bytes(N, V) / 8;
    p.vec = energy_mv_vec(V, D);
    size_t piece = std::min((size_t)V, (size_t)65535 * p.vec);
    if (D * (piece + 1) > words) {
        piece = words / D - 1;
        if (piece > (size_t)p.vec) piece -= piece % p.vec;
    }
    p.piece = (int)piece;
    const int blocks = (p.piece + p.vec - 1) / p.vec;
    const int want = ((D > 2 ? 256 : 512) + blocks - 1) / blocks;
    const int most = std::min((N + 15) / 16, (int)std::min<size_t>(words / (D * (piece + 1)), 1 << 20));
    p.P = std::max(1, std::min(want, most));
    return p;
}

}  // namespace hqa
