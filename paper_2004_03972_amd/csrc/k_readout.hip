// k_readout.hip -- frozen/ambivalent sort, reduced problem, exact enumeration,
// merge and exact Ising energies.
#include <limits.h>
#include <math.h>

#include "exact_acc.h"
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "hqa_internal.h"

namespace hqa {

static_assert(sizeof(Acc256) == ACC_BYTES, "the scratch of the energies is sized by it");

// Position of spin i of replica r in the state arrays.
__device__ __forceinline__ int64_t sidx(int smaj, int ld, int r, int i) {
    return smaj ? (int64_t)i * ld + r : (int64_t)r * ld + i;
}

// ---------------------------------------------------------------------------
// Sort (Results, "Sorting frozen and ambivalent variables"): per replica the n
// spins with the smallest |phibar| (ties: lower index) are ambivalent, listed in
// ascending index; s_i = sgn(phibar_i), sgn(0) = +1.  phibar = S / W in the
// state's precision.  One workgroup (256 threads) per replica: an MSD radix
// select over the bit patterns of |phibar| (non-negative floats order as their
// bit patterns) finds the n-th smallest key K*, then an index-ordered scan takes
// every key < K* and the lowest-index keys == K* up to n.
// ---------------------------------------------------------------------------
struct SelArgs {
    int N, R, ld, smaj, f64, W, n;
    const double *S64;
    const float *S32;
    int32_t *amb;
    int8_t *spins;
    const float *keys;   // if set: keys [R][N] (non-negative) and spins already written
};

__device__ __forceinline__ uint64_t sel_key(const SelArgs &a, int r, int i, int8_t *sgn) {
    if (a.keys) return (uint64_t)__float_as_uint(a.keys[(int64_t)r * a.N + i]);
    if (a.f64) {
        double pb = a.S64[(int64_t)r * a.N + i] / (double)a.W;
        if (sgn) *sgn = pb < 0.0 ? -1 : 1;
        return (uint64_t)__double_as_longlong(fabs(pb));
    }
    float pb = a.S32[sidx(a.smaj, a.ld, r, i)] / (float)a.W;
    if (sgn) *sgn = pb < 0.0f ? -1 : 1;
    return (uint64_t)__float_as_uint(fabsf(pb));
}

// Keys are formed once and kept in LDS where they fit (N <= 8192, or 4096 in binary64); a
// replica-minor state costs a line per value, and workgroups of the 32 replicas of a line run
// on one XCD so that its L2 serves the other 31.  The digit's bin is found by one wavefront, four
// bins a lane.  Measured at N = 4096, R = 1024, replica-minor: 222 us with every pass reading the
// state and one thread walking the bins, 54 us now.
constexpr int SEL_KEYS = 8192;

template <bool KEPT>
__device__ __forceinline__ void select_keys(const SelArgs &a, const int bx_) {
    __shared__ uint32_t hist[256];
    __shared__ uint64_t s_prefix;
    __shared__ int s_k;
    __shared__ int wsum[2][4];
    __shared__ uint64_t s_keys[KEPT ? SEL_KEYS / 2 : 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // workgroup b runs on XCD b mod 8 as a rule: whole groups of 256 replicas are dealt by lines
    const int r = a.smaj && bx_ < (a.R & ~255)
                      ? (bx_ & ~255) + 32 * (bx_ & 7) + ((bx_ >> 3) & 31) : bx_;
    uint32_t *const k32 = (uint32_t *)s_keys;
    auto key = [&](int i) -> uint64_t {
        if constexpr (!KEPT) return sel_key(a, r, i, nullptr);
        return a.f64 ? s_keys[i] : (uint64_t)k32[i];
    };
    // spins
    if (KEPT || !a.keys)
#pragma unroll 4
        for (int i = tid; i < a.N; i += 256) {
            int8_t s;
            const uint64_t k = sel_key(a, r, i, &s);
            if (!a.keys) a.spins[(int64_t)r * a.N + i] = s;
            if (KEPT && a.f64) s_keys[i] = k;
            else if (KEPT) k32[i] = (uint32_t)k;
        }
    if (a.n == 0) return;
    uint64_t prefix = 0, pmask = 0;
    if (tid == 0) s_k = a.n;
    const int passes = a.f64 ? 8 : 4;
    for (int ps = passes - 1; ps >= 0; ps--) {
        hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < a.N; i += 256) {
            uint64_t k = key(i);
            if ((k & pmask) == prefix) atomicAdd(&hist[(k >> (8 * ps)) & 255], 1u);
        }
        __syncthreads();
        if (w == 0) {
            // the bin that holds the k-th key of the prefix (at least k keys have it)
            int c[4], sum = 0;
#pragma unroll
            for (int b = 0; b < 4; b++) {
                c[b] = (int)hist[4 * lane + b];
                sum += c[b];
            }
            int upto = sum;
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(upto, off);
                if (lane >= off) upto += t;
            }
            int k = s_k - (upto - sum);
            if (k >= 1 && k <= sum) {
                int b = 0;
                while (b < 3 && c[b] < k) { k -= c[b]; b++; }
                s_prefix = prefix | ((uint64_t)(4 * lane + b) << (8 * ps));
                s_k = k;
            }
        }
        __syncthreads();
        prefix = s_prefix;
        pmask |= (uint64_t)255 << (8 * ps);
    }
    const uint64_t kstar = prefix;
    const int m = s_k;  // how many keys equal to K* are taken
    int eq_run = 0, out_run = 0;
    for (int c0 = 0; c0 < a.N; c0 += 256) {
        int i = c0 + tid;
        uint64_t k = i < a.N ? key(i) : ~0ull;
        bool eq = i < a.N && k == kstar;
        bool lt = i < a.N && k < kstar;
        uint64_t beq = __ballot(eq);
        uint64_t lanemask = lane ? (~0ull >> (64 - lane)) : 0ull;
        int eq_before_w = __popcll(beq & lanemask);
        if (lane == 0) wsum[0][w] = __popcll(beq);
        __syncthreads();
        int eq_before = eq_run + eq_before_w;
        for (int v = 0; v < w; v++) eq_before += wsum[0][v];
        bool sel = lt || (eq && eq_before < m);
        uint64_t bsel = __ballot(sel);
        if (lane == 0) wsum[1][w] = __popcll(bsel);
        __syncthreads();
        int pos = out_run + __popcll(bsel & lanemask);
        for (int v = 0; v < w; v++) pos += wsum[1][v];
        if (sel && pos < a.n) a.amb[(int64_t)r * a.n + pos] = i;
        for (int v = 0; v < 4; v++) { eq_run += wsum[0][v]; out_run += wsum[1][v]; }
        __syncthreads();
    }
}

__device__ __forceinline__ void select_body(const SelArgs &a, const int bx_) {
    if (a.N <= (a.f64 ? SEL_KEYS / 2 : SEL_KEYS)) select_keys<true>(a, bx_);
    else select_keys<false>(a, bx_);
}

__global__ __launch_bounds__(256) void k_select(SelArgs a) { select_body(a, blockIdx.x); }

// Many instances in one launch: instance blockIdx.y, its own block count nb[y].
__global__ __launch_bounds__(256) void k_select_many(const SelArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const SelArgs a = as[k];
    select_body(a, blockIdx.x);
}

hipError_t launch_select(const Instance &I, int R, int prec, int W, int n, int32_t *amb,
                         int8_t *spins, hipStream_t st) {
    SelArgs a;
    a.N = I.N; a.R = R; a.ld = I.ld; a.smaj = I.smaj; a.f64 = prec == HQA_PREC_F64_REF;
    a.W = W; a.n = n; a.S64 = I.S64; a.S32 = I.S32; a.amb = amb; a.spins = spins;
    a.keys = nullptr;
    k_select<<<R, 256, 0, st>>>(a);
    return hipGetLastError();
}

// Selection on explicit keys (ascending, ties to the lower index); spins untouched.
hipError_t launch_select_keys(int N, int R, const float *keys, int n, int32_t *amb,
                              int8_t *spins, hipStream_t st) {
    SelArgs a;
    a.N = N; a.R = R; a.ld = N; a.smaj = 0; a.f64 = 0; a.W = 1; a.n = n;
    a.S64 = nullptr; a.S32 = nullptr; a.amb = amb; a.spins = spins; a.keys = keys;
    k_select<<<R, 256, 0, st>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Reduced problem (HQA section, effective couplings): J_eff = J[A, A] and
// h_eff_a = h_a + sum_{k not in A} J_ak s_k, each h_eff the correctly rounded
// exact sum.  One wavefront per (replica, ambivalent spin).
// ---------------------------------------------------------------------------
struct RedArgs {
    int N, R, n, csr, b0;
    int words;            // 32-bit words of the dense sums (see reduce_words), 0: one accumulator
    double scale;         // 2^-b0
    const double *J;
    const int32_t *rp, *ci;
    const double *h;
    const int32_t *amb;
    const int8_t *spins;
    double *h_eff, *J_eff;
};

__device__ __forceinline__ bool in_sorted(const int32_t *A, int n, int k) {
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (A[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo < n && A[lo] == k;
}

__device__ __forceinline__ double jlookup(const RedArgs &a, int i, int j) {
    if (!a.csr) return a.J[(int64_t)i * a.N + j];
    int lo = a.rp[i], hi = a.rp[i + 1];
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a.ci[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    return (lo < a.rp[i + 1] && a.ci[lo] == j) ? a.J[lo] : 0.0;
}

// x 2^-b0 s added to W sums: the integer in W words from the top, adding 1.5 2^52 rounds to an
// integer and fma takes it off exactly, so that every sum of them is exact in binary64.
template <int W>
__device__ __forceinline__ void words_add(double x, double s, double scale, double (&sum)[W]) {
    constexpr double RND = 0x1.8p52;
    double m = x * scale;
    if constexpr (W > 2) {
        const double h = __builtin_fma(m, 0x1p-64, RND) - RND;
        m = __builtin_fma(h, -0x1p64, m);
        sum[2] = __builtin_fma(h, s, sum[2]);
    }
    if constexpr (W > 1) {
        const double h = __builtin_fma(m, 0x1p-32, RND) - RND;
        m = __builtin_fma(h, -0x1p32, m);
        sum[1] = __builtin_fma(h, s, sum[1]);
    }
    sum[0] = __builtin_fma(m, s, sum[0]);
}

// acc += sum over k not in A of J_k s_k, on lane 0: every k, then the ambivalent ones taken off
// (both exact).
template <int W>
__device__ __forceinline__ void reduce_row(const RedArgs &a, const double *Jr, const int8_t *s,
                                           const int32_t *A, int lane, Acc256 &acc) {
    double sum[W];
#pragma unroll
    for (int w = 0; w < W; w++) sum[w] = 0.0;
#pragma unroll 8
    for (int k = lane; k < a.N; k += 64) words_add<W>(Jr[k], (double)s[k], a.scale, sum);
    for (int b = lane; b < a.n; b += 64) {
        const int k = A[b];
        if (k >= 0 && k < a.N) words_add<W>(Jr[k], -(double)s[k], a.scale, sum);
    }
#pragma unroll
    for (int w = 0; w < W; w++) {
        for (int o = 32; o > 0; o >>= 1) sum[w] += __shfl_xor(sum[w], o);
        if (lane == 0) acc_add(acc, ldexp(sum[w], a.b0 + 32 * w), a.b0);
    }
}

// Bound by the reads of J's rows.  n = 20, R = 64, 24 instances of 500 to 5000 spins: 509 us with
// a fixed-point accumulator a lane and a search of A for every k, 140 us with sums of words.
__device__ __forceinline__ void reduce_body(const RedArgs &a, const int bx_) {
    const int lane = threadIdx.x & 63;
    const int64_t wid = ((int64_t)bx_ * blockDim.x + threadIdx.x) >> 6;
    if (wid >= (int64_t)a.R * a.n) return;
    const int r = (int)(wid / a.n), ai = (int)(wid % a.n);
    const int32_t *A = a.amb + (int64_t)r * a.n;
    const int8_t *s = a.spins + (int64_t)r * a.N;
    const int row = A[ai];
    if (row < 0 || row >= a.N) return;
    Acc256 acc;
    acc_zero(acc);
    if (lane == 0) acc_add(acc, a.h[row], a.b0);
    const double *Jr = a.J + (int64_t)row * a.N;
    if (a.words == 1) {
        reduce_row<1>(a, Jr, s, A, lane, acc);
    } else if (a.words == 2) {
        reduce_row<2>(a, Jr, s, A, lane, acc);
    } else if (a.words == 3) {
        reduce_row<3>(a, Jr, s, A, lane, acc);
    } else if (!a.csr) {
        for (int k = lane; k < a.N; k += 64)
            if (!in_sorted(A, a.n, k)) acc_add(acc, Jr[k] * (double)s[k], a.b0);
    } else {
        for (int e = a.rp[row] + lane; e < a.rp[row + 1]; e += 64) {
            int k = a.ci[e];
            if (!in_sorted(A, a.n, k)) acc_add(acc, a.J[e] * (double)s[k], a.b0);
        }
    }
    acc_wave_allreduce(acc);
    if (lane == 0) a.h_eff[(int64_t)r * a.n + ai] = acc_round(acc, a.b0);
    if (a.J_eff)   // optional: the tabu search reads J[A, A] from the instance itself
        for (int b = lane; b < a.n; b += 64)
            a.J_eff[((int64_t)r * a.n + ai) * a.n + b] = jlookup(a, row, A[b]);
}

__global__ __launch_bounds__(256) void k_reduce(RedArgs a) { reduce_body(a, blockIdx.x); }

__global__ __launch_bounds__(256) void k_reduce_many(const RedArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const RedArgs a = as[k];
    reduce_body(a, blockIdx.x);
}

// Words of the dense sums: the N + n terms below 2^span leave every sum of the top words
// below 2^53, and those of 32-bit words (rounded, up to 2^31) too.  0 for CSR rows, wider spans
// and scales near binary64's range.
static int reduce_words(const Instance &I, int n) {
    if (I.layout == HQA_CSR || I.es.lsb == INT32_MIN) return 0;
    if (I.es.msb > 900 || I.es.lsb < -900 || I.N > (1 << 20)) return 0;
    const int span = I.es.msb + 1 - I.es.lsb;
    int lg = 1;
    while (((int64_t)1 << lg) < (int64_t)I.N + n) lg++;
    for (int w = 1; w <= 3; w++)
        if (span - 32 * (w - 1) + lg <= 53) return w;
    return 0;
}

hipError_t launch_reduce(const Instance &I, int R, int n, const int32_t *amb,
                         const int8_t *spins, double *h_eff, double *J_eff, hipStream_t st) {
    RedArgs a;
    a.N = I.N; a.R = R; a.n = n; a.csr = I.layout == HQA_CSR; a.b0 = I.es.lsb;
    a.words = reduce_words(I, n);
    a.scale = a.words ? std::ldexp(1.0, -I.es.lsb) : 0.0;
    a.J = I.J64; a.rp = I.rp; a.ci = I.ci; a.h = I.h64;
    a.amb = amb; a.spins = spins; a.h_eff = h_eff; a.J_eff = J_eff;
    int64_t waves = (int64_t)R * n;
    if (waves == 0) return hipSuccess;
    k_reduce<<<(unsigned)((waves + 3) / 4), 256, 0, st>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exact minimum of the reduced energy E'(c) = sum_{a<b} J_ab x_a x_b + sum_a h_a x_a
// over all codes c (bit a set: x_a = -1), ties to the smallest code.  Thread t
// fixes the top bits of the code to t and walks the low bits (one workgroup per replica
// for integer couplings, several for real ones; see k_enumerate_int and k_enum_real),
// updating E' and the local fields f_a = h_a + sum_{b != a} J_ab x_b by flips
// (dE = -2 x_a f_a).  Integer instances run in int32 or int64 (exact).  Otherwise pass 1
// walks in binary64 and pass 2 re-walks, rescoring exactly (fixed-point accumulator,
// rounded once) every code whose binary64 energy lies within a rigorous error bound of
// the pass-1 minimum.
// ---------------------------------------------------------------------------
#define ENUM_MAXN 24
#define ENERGY_MAXN_LDS 16384
#define ENUM_MAXLOW 16

template <typename T>
struct EnumState {
    T E;
    int64_t code;
};

__device__ __forceinline__ bool better_i(int64_t e1, int64_t c1, int64_t e2, int64_t c2) {
    return e1 < e2 || (e1 == e2 && c1 < c2);
}
__device__ __forceinline__ bool better_d(double e1, int64_t c1, double e2, int64_t c2) {
    return e1 < e2 || (e1 == e2 && c1 < c2);
}

struct EnumArgs {
    int n, R, b0, integral;
    const double *J_eff, *h_eff;
    int64_t *code;
    double *e_red;
};

template <typename T>
__device__ __forceinline__ T energy_from_scratch(const T *J, const T *h, int n, uint32_t code) {
    T E = 0;
    for (int a = 0; a < n; a++) {
        T xa = ((code >> a) & 1) ? (T)-1 : (T)1;
        T acc = 0;
        for (int b = a + 1; b < n; b++) {
            T xb = ((code >> b) & 1) ? (T)-1 : (T)1;
            acc = acc + J[a * n + b] * xb;
        }
        E = E + xa * (acc + h[a]);
    }
    return E;
}

__device__ __forceinline__ double energy_exact(const double *J, const double *h, int n,
                                               uint32_t code, int b0) {
    Acc256 acc;
    acc_zero(acc);
    for (int a = 0; a < n; a++) {
        double xa = ((code >> a) & 1) ? -1.0 : 1.0;
        for (int b = a + 1; b < n; b++) {
            double xb = ((code >> b) & 1) ? -1.0 : 1.0;
            acc_add(acc, J[a * n + b] * (xa * xb), b0);
        }
        acc_add(acc, h[a] * xa, b0);
    }
    return acc_round(acc, b0);
}

// Gray walk over the low `nl` bits with the top bits fixed to `top`.  The visitor
// sees (energy, code) for every code of the chunk.
template <typename T, typename Visit>
__device__ __forceinline__ void gray_walk(const T *J, const T *h, int n, int nl, uint32_t top,
                                          T *f, Visit visit) {
    uint32_t code = top << nl;
    T E = energy_from_scratch<T>(J, h, n, code);
    for (int a = 0; a < nl; a++) {
        T acc = h[a];
        for (int b = 0; b < n; b++)
            if (b != a) acc = acc + J[a * n + b] * (((code >> b) & 1) ? (T)-1 : (T)1);
        f[a] = acc;
    }
    visit(E, code);
    const uint32_t cnt = 1u << nl;
    for (uint32_t k = 1; k < cnt; k++) {
        int a = __ffs(k) - 1;
        T xa = ((code >> a) & 1) ? (T)-1 : (T)1;
        E = E - (T)2 * xa * f[a];
        for (int b = 0; b < nl; b++)
            if (b != a) f[b] = f[b] - (T)2 * J[a * n + b] * xa;
        code ^= 1u << a;
        visit(E, code);
    }
}

// Real couplings, many codes: the code space of each replica is split over P
// workgroups of 256 threads; thread t of workgroup p fixes the top pt = n - NL bits of
// the code to p * 256 + t and walks the NL low bits by blocks as k_enumerate_int does: E and
// the fields from scratch at the start (m and 2 n roundings), one rounding of E and of each
// field per flip between blocks, and within a block at most nine for a code's change of E (a
// sum of up to four fields, each within 2 n + K / 8 roundings by then, and of up to six
// couplings).  All are of numbers within 4 S, and K / 16 flips leave the errors below the
// bound u S (m + K (2 n + 1) + K^2) of a walk that flips K = 2^NL times.
//   k_enum_real<NL, 1>: each workgroup's binary64 minimum -> part;
//   k_enum_real_mid: per replica, the minimum over the workgroups and the rescoring
//     threshold E_min + 2 delta + 4 u S (the bound of k_enumerate);
//   k_enum_real<NL, 2>: workgroups whose minimum is at or below the threshold walk again and
//     collect every such code, which a wavefront each then rescores exactly (fixed-point
//     accumulator, rounded once); each workgroup's exact minimum -> part;
//   k_enum_real_mid: per replica, the exact minimum over the workgroups, ties to the
//     smallest code.
// Bound by binary64 additions in pass 1 (three a code), the exact sums in pass 2.  n = 20,
// 64 replicas of 12 instances: 836 us a pass with the code kept beside each minimum and both
// walks in full; now 270 us for pass 1 (456 with every field updated per code), 65 for pass 2
// (255 with each candidate's terms added by the thread that found it).
// ---------------------------------------------------------------------------
#define ENUM_PT_REAL 12
#define ENUM_CAND 256    // candidates a workgroup rescores together; further ones by their thread

struct EnumRealArgs {
    int n, R, P, b0;
    const double *J_eff, *h_eff;
    double *partE;        // [R][P]
    int64_t *partC;       // [R][P]
    double *thresh;       // [R]
    int64_t *code;
    double *e_red;
};

template <int NL, int PASS>
__device__ __forceinline__ void enum_real_body(const EnumRealArgs &a, const int bx_) {
    __shared__ double Jd[ENUM_MAXN * ENUM_MAXN], J4[ENUM_MAXN * ENUM_MAXN], hd[ENUM_MAXN];
    __shared__ double sE[256];
    __shared__ int64_t sC[PASS == 2 ? 256 : 1];
    __shared__ uint32_t cand[PASS == 2 ? ENUM_CAND : 1];   // codes to rescore
    __shared__ int ncand;
    const int r = bx_ / a.P, p = bx_ % a.P, tid = threadIdx.x, n = a.n;
    const double thr = PASS == 2 ? a.thresh[r] : 0.0;
    // pass 2 walks the same binary64 energies: without one at or below the threshold in pass 1
    // this workgroup has no code to rescore
    if (PASS == 2 && !(a.partE[(int64_t)r * a.P + p] <= thr)) {
        __syncthreads();
        if (tid == 0) {
            a.partE[(int64_t)r * a.P + p] = INFINITY;
            a.partC[(int64_t)r * a.P + p] = INT64_MAX;
        }
        return;
    }
    for (int k = tid; k < n * n; k += 256) {
        const double v = a.J_eff[(int64_t)r * n * n + k];
        Jd[k] = v;
        J4[k / n * ENUM_MAXN + k % n] = 4.0 * v;
    }
    for (int k = tid; k < n; k += 256) hd[k] = a.h_eff[(int64_t)r * n + k];
    if (PASS == 2 && tid == 0) ncand = 0;
    __syncthreads();
    const uint32_t top = (uint32_t)(p * 256 + tid);
    const bool active = top < (1u << (n - NL));
    double bestE = INFINITY;
    int64_t bestC = INT64_MAX;
    if (active) {
        const uint32_t code = top << NL;
        double E = energy_from_scratch<double>(Jd, hd, n, code);
        constexpr int NA = NL < 4 ? NL : 4, NC = 1 << NA, NBLK = 1 << (NL - NA), NU = NBLK < 4 ? NBLK : 4;
        // G_b = -2 f_b with the block's bits 0: flipping b from there adds G_b x_b
        double G[NL ? NL : 1], Q[NC];
#pragma unroll
        for (int aa = 0; aa < NL; aa++) {
            double acc = hd[aa];
            for (int b = 0; b < n; b++)
                if (b != aa) acc = acc + Jd[aa * n + b] * (((code >> b) & 1) ? -1.0 : 1.0);
            G[aa] = -2.0 * acc;
        }
        // pairs flipped together, by code of the block
#pragma unroll
        for (int c = 0; c < NC; c++) {
            Q[c] = 0.0;
#pragma unroll
            for (int x = 0; x < NA; x++)
#pragma unroll
                for (int y = x + 1; y < NA; y++)
                    if ((c >> x & 1) && (c >> y & 1)) Q[c] = Q[c] + J4[x * ENUM_MAXN + y];
        }
        uint32_t up = 0;                               // the low bits above the block's, uniform
        auto block = [&]() {
            double u[NC], mn = 0.0;
            u[0] = 0.0;
#pragma unroll
            for (int c = 1; c < NC; c++) {
                const int t = 31 - __builtin_clz(c), c0 = c ^ (1 << t);
                u[c] = c0 ? u[c0] + G[t] : G[t];       // sum of G over the flipped bits
            }
#pragma unroll
            for (int c = 1; c < NC; c++) {
                if (c & (c - 1)) u[c] = u[c] + Q[c];
                mn = __builtin_fmin(mn, u[c]);
            }
            // rounding is monotone: E + mn is the least of the block's E + u
            if constexpr (PASS == 1) {
                bestE = __builtin_fmin(bestE, E + mn);
            } else if (E + mn <= thr) {
#pragma unroll 1
                for (int c = 0; c < NC; c++) {
                    double uc = u[0];
#pragma unroll
                    for (int k = 1; k < NC; k++) uc = k == c ? u[k] : uc;
                    if (E + uc <= thr) {
                        const uint32_t full = code | up | (uint32_t)c;
                        const int slot = atomicAdd(&ncand, 1);
                        if (slot < ENUM_CAND) {
                            cand[slot] = full;
                            continue;
                        }
                        const double ex = energy_exact(Jd, hd, n, full, a.b0);
                        if (better_d(ex, full, bestE, bestC)) { bestE = ex; bestC = full; }
                    }
                }
            }
        };
        // flip of bit aa (uniform), x_a +1 where its bit is 0
        auto flip = [&](int aa, double ga, const double (&row)[NL ? NL : 1]) {
            const double xa = ((up >> aa) & 1u) ? -1.0 : 1.0;
            E = __builtin_fma(xa, ga, E);
#pragma unroll
            for (int b = 0; b < NL; b++) G[b] = __builtin_fma(xa, row[b], G[b]);   // J_aa = 0
            up ^= 1u << aa;
        };
        if constexpr (NL > 4) {
            double R4[NL], R5[NL];
#pragma unroll
            for (int b = 0; b < NL; b++) {
                R4[b] = J4[4 * ENUM_MAXN + b];
                R5[b] = NL > 5 ? J4[5 * ENUM_MAXN + b] : 0.0;
            }
            for (int m = 0; m < NBLK; m += NU) {
                block();
                flip(4, G[4], R4);
                block();
                if constexpr (NL > 5) {
                    flip(5, G[5], R5);
                    block();
                    flip(4, G[4], R4);
                    block();
                    if (m + NU < NBLK) {
                        const int aa = 4 + __builtin_ctz(m + NU);
                        double ga = G[0], row[NL];
#pragma unroll
                        for (int b = 6; b < NL; b++) ga = b == aa ? G[b] : ga;
#pragma unroll
                        for (int b = 0; b < NL; b++) row[b] = J4[aa * ENUM_MAXN + b];
                        flip(aa, ga, row);
                    }
                }
            }
        } else {
            block();
        }
    }
    if constexpr (PASS == 2) {
        // a wavefront a candidate, its terms over the lanes (exact sums have no order)
        __syncthreads();
        const int lane = tid & 63, total = min(ncand, ENUM_CAND);
        for (int k = tid >> 6; k < total; k += 4) {
            const uint32_t c = cand[k];
            Acc256 acc;
            acc_zero(acc);
            for (int t = lane; t < n * n; t += 64) {
                const int x = t / n, y = t % n;
                const double sx = ((c >> x) & 1) ? -1.0 : 1.0, sy = ((c >> y) & 1) ? -1.0 : 1.0;
                if (y >= x) acc_add(acc, y > x ? Jd[t] * (sx * sy) : hd[x] * sx, a.b0);
            }
            acc_wave_allreduce(acc);
            const double ex = acc_round(acc, a.b0);
            if (lane == 0 && better_d(ex, c, bestE, bestC)) { bestE = ex; bestC = c; }
        }
    }
    sE[tid] = bestE;
    if (PASS == 2) sC[tid] = bestC;
    __syncthreads();
    for (int s2 = 128; s2 > 0; s2 >>= 1) {
        if (tid < s2) {
            if constexpr (PASS == 1) {
                if (sE[tid + s2] < sE[tid]) sE[tid] = sE[tid + s2];
            } else if (better_d(sE[tid + s2], sC[tid + s2], sE[tid], sC[tid])) {
                sE[tid] = sE[tid + s2];
                sC[tid] = sC[tid + s2];
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        a.partE[(int64_t)r * a.P + p] = sE[0];
        a.partC[(int64_t)r * a.P + p] = PASS == 2 ? sC[0] : 0;
    }
}

template <int NL, int PASS>
__global__ __launch_bounds__(256) void k_enum_real(EnumRealArgs a) {
    enum_real_body<NL, PASS>(a, blockIdx.x);
}

template <int NL, int PASS>
__global__ __launch_bounds__(256) void k_enum_real_many(const EnumRealArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const EnumRealArgs a = as[k];
    enum_real_body<NL, PASS>(a, blockIdx.x);
}

// One wavefront per replica: minimum over the P workgroup results; after pass 1 the
// rescoring threshold, after pass 2 the result.
__device__ __forceinline__ void enum_real_mid_body(const EnumRealArgs &a, int pass, const int bx_) {
    const int r = bx_, lane = threadIdx.x, n = a.n;
    double E = INFINITY;
    int64_t C = INT64_MAX;
    for (int p = lane; p < a.P; p += 64) {
        const double e2 = a.partE[(int64_t)r * a.P + p];
        const int64_t c2 = a.partC[(int64_t)r * a.P + p];
        if (better_d(e2, c2, E, C)) { E = e2; C = c2; }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double e2 = __shfl_xor(E, off);
        const int64_t c2 = __shfl_xor(C, off);
        if (better_d(e2, c2, E, C)) { E = e2; C = c2; }
    }
    if (pass == 2) {
        if (lane == 0) {
            a.code[r] = C;
            a.e_red[r] = E;
        }
        return;
    }
    // rigorous bound on |E_binary64 - E_exact| along a walk of K = 2^NL codes:
    // u S (m + K (2n + 1) + K^2) with S = sum |J_ab| (a < b) + sum |h_a|, m the term
    // count, u = 2^-53; doubled (the minimum's own error and a candidate's), plus the
    // rounding of the exact values themselves
    double Ssum = 0.0;
    const double *J = a.J_eff + (int64_t)r * n * n, *h = a.h_eff + (int64_t)r * n;
    for (int k = lane; k < n * n; k += 64)
        if (k % n > k / n) Ssum += fabs(J[k]);
    for (int k = lane; k < n; k += 64) Ssum += fabs(h[k]);
    for (int off = 32; off > 0; off >>= 1) Ssum += __shfl_xor(Ssum, off);
    if (lane == 0) {
        const int nl = n > ENUM_PT_REAL ? n - ENUM_PT_REAL : 0;
        const double S = Ssum * (1.0 + 1e-12);
        const double K = (double)(1u << nl);
        const double mterms = (double)(n * (n - 1) / 2 + n);
        const double u = 1.1102230246251565e-16;
        const double delta = u * S * (mterms + K * (2.0 * n + 1.0) + K * K);
        a.thresh[r] = E + 2.0 * delta + 4.0 * u * S;
    }
}

__global__ __launch_bounds__(64) void k_enum_real_mid(EnumRealArgs a, int pass) {
    enum_real_mid_body(a, pass, blockIdx.x);
}

__global__ __launch_bounds__(64) void k_enum_real_mid_many(const EnumRealArgs *as, const int *nb,
                                                          int pass) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const EnumRealArgs a = as[k];
    enum_real_mid_body(a, pass, blockIdx.x);
}

template <int NL>
static void launch_enum_real(const EnumRealArgs &a, hipStream_t st) {
    k_enum_real<NL, 1><<<a.R * a.P, 256, 0, st>>>(a);
    k_enum_real_mid<<<a.R, 64, 0, st>>>(a, 1);
    k_enum_real<NL, 2><<<a.R * a.P, 256, 0, st>>>(a);
    k_enum_real_mid<<<a.R, 64, 0, st>>>(a, 2);
}

size_t enum_scratch_bytes(int n, int R) {
    const int pt = n < ENUM_PT_REAL ? n : ENUM_PT_REAL;
    const int P = ((1 << pt) + 255) / 256;
    return (size_t)R * P * 16 + (size_t)R * 8 + 64;
}

// Integer instances with small sums: 1024 threads per replica, thread t fixes the
// top pt = n - NL <= 10 bits of the code to t and walks the NL low bits in int32: blocks of
// the 16 codes of the lowest four bits, one flip of a higher bit (Gray order) between them.
// From the block's first code, all four x = +1, flipping the set F changes E' by
// -2 sum_F f_a + 4 sum_{a<b in F} J_ab; the second sum is the replica's, so a code costs an
// addition, a 24-bit multiply-add and a minimum, and only the flips between blocks update the
// NL fields.  The low bits of every thread follow the same sequence, so the flipped bit and
// its sign are wavefront-uniform.  The walk keeps the minimum of the key
// (E' + S) << NL | low code, so equal energies resolve to the smallest code.
// Requires every |J_ab|, |h_a| integral with S = sum_{a<b} |J_ab| + sum_a |h_a| below
// 2^22 and 2 S < 2^(31 - NL) (sums of f over F stay within 2 S, changes of E' within 2 S: all
// terms then fit the 24-bit products and the key); other integer replicas take the int64 walk.
// Measured at n = 20, R = 1024: 440 us with every field updated per code, 233 this way.
#define ENUM_PT 10

__device__ __forceinline__ int32_t mad24(int32_t x, int32_t y, int32_t z) {
    return __mul24(x, y) + z;
}

template <int NL>
__device__ __forceinline__ void walk_i32(const int32_t *Jv, const int32_t *J2, const int32_t *hv,
                                         int n, uint32_t top, int32_t S, int64_t &bestE,
                                         int64_t &bestC) {
    // start: low bits all 0 (x = +1), top bits from `top`
    auto xof = [&](int c) -> int32_t {
        return c < NL ? 1 : (((top >> (c - NL)) & 1u) ? -1 : 1);
    };
    int32_t E = S;
    for (int aa = 0; aa < n; aa++) {
        int32_t acc = hv[aa];
        for (int bb = aa + 1; bb < n; bb++) acc += Jv[aa * n + bb] * xof(bb);
        E += xof(aa) * acc;
    }
    constexpr int NA = NL < 4 ? NL : 4, NC = 1 << NA, NBLK = 1 << (NL - NA), NU = NBLK < 4 ? NBLK : 4;
    int32_t f[NL ? NL : 1], Q[NC];
#pragma unroll
    for (int b = 0; b < NL; b++) {
        int32_t acc = hv[b];
        for (int c = 0; c < n; c++) acc += Jv[b * n + c] * xof(c);   // J_bb = 0
        f[b] = acc;
    }
    // pairs flipped together, by code of the block, with that code below them
#pragma unroll
    for (int c = 0; c < NC; c++) {
        int32_t t = 0;
#pragma unroll
        for (int x = 0; x < NA; x++)
#pragma unroll
            for (int y = x + 1; y < NA; y++)
                if ((c >> x & 1) && (c >> y & 1)) t += 2 * J2[x * ENUM_MAXN + y];
        Q[c] = (int32_t)((uint32_t)t << NL) + c;
    }
    uint32_t g = 0, key = 0xffffffffu;                 // g: the low bits above the block's, uniform
    auto block = [&]() {
        int32_t u[NC], mn = 0;
#pragma unroll
        for (int c = 1; c < NC; c++) {
            const int t = 31 - __builtin_clz(c), c0 = c ^ (1 << t);
            u[c] = c0 ? u[c0] + f[t] : f[t];           // sum of f over the flipped bits
        }
#pragma unroll
        for (int c = 1; c < NC; c++) mn = min(mn, mad24(u[c], -(2 << NL), Q[c]));
        key = min(key, ((uint32_t)E << NL) + g + (uint32_t)mn);
    };
    auto flip = [&](int aa, int32_t fa, const int32_t (&row)[NL ? NL : 1]) {
        const int32_t sgn = ((g >> aa) & 1u) ? 1 : -1;   // -x_a before the flip
        E = mad24(fa, 2 * sgn, E);
#pragma unroll
        for (int b = 0; b < NL; b++) f[b] = mad24(row[b], sgn, f[b]);   // J_aa = 0
        g ^= 1u << aa;
    };
    if constexpr (NL > 4) {
        int32_t R4[NL], R5[NL];
#pragma unroll
        for (int b = 0; b < NL; b++) {
            R4[b] = J2[4 * ENUM_MAXN + b];
            R5[b] = NL > 5 ? J2[5 * ENUM_MAXN + b] : 0;
        }
        for (int m = 0; m < NBLK; m += NU) {
            block();
            flip(4, f[4], R4);
            block();
            if constexpr (NL > 5) {
                flip(5, f[5], R5);
                block();
                flip(4, f[4], R4);
                block();
                if (m + NU < NBLK) {
                    const int aa = 4 + __builtin_ctz(m + NU);
                    int32_t fa = f[0], row[NL];
#pragma unroll
                    for (int b = 6; b < NL; b++) fa = b == aa ? f[b] : fa;
#pragma unroll
                    for (int b = 0; b < NL; b++) row[b] = J2[aa * ENUM_MAXN + b];
                    flip(aa, fa, row);
                }
            }
        }
    } else {
        block();
    }
    bestE = (int64_t)(key >> NL) - S;
    bestC = ((int64_t)top << NL) | (key & ((1u << NL) - 1u));
}

template <int NL>
__device__ __forceinline__ void enumerate_int_body(const EnumArgs &a, const int bx_) {
    __shared__ int32_t Jv[ENUM_MAXN * ENUM_MAXN], J2[ENUM_MAXN * ENUM_MAXN], hv[ENUM_MAXN];
    __shared__ int64_t Jl[ENUM_MAXN * ENUM_MAXN], hl[ENUM_MAXN];
    __shared__ int64_t sEi[1024], sC[1024];
    __shared__ unsigned long long sS;
    const int r = bx_, tid = threadIdx.x, n = a.n;
    if (tid == 0) sS = 0;
    __syncthreads();
    for (int k = tid; k < n * n; k += 1024) {
        const int64_t v = (int64_t)a.J_eff[(int64_t)r * n * n + k];
        Jl[k] = v;
        if (k / n < k % n) atomicAdd(&sS, (unsigned long long)(v < 0 ? -v : v));
    }
    for (int k = tid; k < n; k += 1024) {
        const int64_t v = (int64_t)a.h_eff[(int64_t)r * n + k];
        hl[k] = v;
        atomicAdd(&sS, (unsigned long long)(v < 0 ? -v : v));
    }
    __syncthreads();
    const unsigned long long S = sS;
    const bool fast = S < (1ull << 22) && 2 * S < (1ull << (31 - NL));   // uniform
    if (fast) {
        for (int k = tid; k < n * n; k += 1024) {
            Jv[k] = (int32_t)Jl[k];
            J2[k / n * ENUM_MAXN + k % n] = 2 * (int32_t)Jl[k];
        }
        for (int k = tid; k < n; k += 1024) hv[k] = (int32_t)hl[k];
        __syncthreads();
    }
    const bool active = tid < (1 << (n - NL));
    int64_t bestE = INT64_MAX, bestC = INT64_MAX;
    if (active) {
        if (fast) {
            walk_i32<NL>(Jv, J2, hv, n, (uint32_t)tid, (int32_t)S, bestE, bestC);
        } else {
            int64_t f[ENUM_MAXLOW];
            gray_walk<int64_t>(Jl, hl, n, NL, (uint32_t)tid, f, [&](int64_t E, uint32_t c) {
                if (better_i(E, c, bestE, bestC)) { bestE = E; bestC = c; }
            });
        }
    }
    // argmin over the workgroup, ties to the smaller code
    sEi[tid] = bestE;
    sC[tid] = bestC;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if (tid < st && better_i(sEi[tid + st], sC[tid + st], sEi[tid], sC[tid])) {
            sEi[tid] = sEi[tid + st];
            sC[tid] = sC[tid + st];
        }
        __syncthreads();
    }
    if (tid == 0) {
        a.code[r] = sC[0];
        a.e_red[r] = (double)sEi[0];
    }
}

template <int NL>
__global__ __launch_bounds__(1024) void k_enumerate_int(EnumArgs a) {
    enumerate_int_body<NL>(a, blockIdx.x);
}

template <int NL>
__global__ __launch_bounds__(1024) void k_enumerate_int_many(const EnumArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const EnumArgs a = as[k];
    enumerate_int_body<NL>(a, blockIdx.x);
}

template <int NL>
static void launch_enum_int(const EnumArgs &a, hipStream_t st) {
    k_enumerate_int<NL><<<a.R, 1024, 0, st>>>(a);
}

hipError_t launch_enumerate(int n, int R, const double *J_eff, const double *h_eff, int b0,
                            int integral, int64_t *code, double *e_red, void *scratch,
                            hipStream_t st) {
    EnumArgs a;
    a.n = n; a.R = R; a.b0 = b0; a.integral = integral;
    a.J_eff = J_eff; a.h_eff = h_eff; a.code = code; a.e_red = e_red;
    if (R == 0) return hipSuccess;
    if (!integral) {
        EnumRealArgs b;
        const int pt = n < ENUM_PT_REAL ? n : ENUM_PT_REAL;
        b.n = n; b.R = R; b.P = ((1 << pt) + 255) / 256; b.b0 = b0;
        b.J_eff = J_eff; b.h_eff = h_eff; b.code = code; b.e_red = e_red;
        b.partE = (double *)scratch;
        b.partC = (int64_t *)((char *)scratch + (size_t)R * b.P * 8);
        b.thresh = (double *)((char *)scratch + (size_t)R * b.P * 16);
        switch (n - pt) {
            case 0: launch_enum_real<0>(b, st); break;
            case 1: launch_enum_real<1>(b, st); break;
            case 2: launch_enum_real<2>(b, st); break;
            case 3: launch_enum_real<3>(b, st); break;
            case 4: launch_enum_real<4>(b, st); break;
            case 5: launch_enum_real<5>(b, st); break;
            case 6: launch_enum_real<6>(b, st); break;
            case 7: launch_enum_real<7>(b, st); break;
            case 8: launch_enum_real<8>(b, st); break;
            case 9: launch_enum_real<9>(b, st); break;
            case 10: launch_enum_real<10>(b, st); break;
            case 11: launch_enum_real<11>(b, st); break;
            default: launch_enum_real<12>(b, st); break;
        }
        return hipGetLastError();
    }
    switch (n > ENUM_PT ? n - ENUM_PT : 0) {   // low bits walked per thread
        case 0: launch_enum_int<0>(a, st); break;
        case 1: launch_enum_int<1>(a, st); break;
        case 2: launch_enum_int<2>(a, st); break;
        case 3: launch_enum_int<3>(a, st); break;
        case 4: launch_enum_int<4>(a, st); break;
        case 5: launch_enum_int<5>(a, st); break;
        case 6: launch_enum_int<6>(a, st); break;
        case 7: launch_enum_int<7>(a, st); break;
        case 8: launch_enum_int<8>(a, st); break;
        case 9: launch_enum_int<9>(a, st); break;
        case 10: launch_enum_int<10>(a, st); break;
        case 11: launch_enum_int<11>(a, st); break;
        case 12: launch_enum_int<12>(a, st); break;
        case 13: launch_enum_int<13>(a, st); break;
        default: launch_enum_int<14>(a, st); break;
    }
    return hipGetLastError();
}

struct MergeArgs {
    int N, R, n;
    const int32_t *amb;
    const int64_t *code;
    int8_t *spins;
};

__device__ __forceinline__ void merge_body(int N, int R, int n, const int32_t *amb,
                                           const int64_t *code, int8_t *spins, const int bx_) {
    int64_t t = (int64_t)bx_ * blockDim.x + threadIdx.x;
    if (t >= (int64_t)R * n) return;
    int r = (int)(t / n), ai = (int)(t % n);
    int i = amb[t];
    if (i < 0 || i >= N) return;
    spins[(int64_t)r * N + i] = ((code[r] >> ai) & 1) ? -1 : 1;
}

__global__ void k_merge(int N, int R, int n, const int32_t *amb, const int64_t *code,
                        int8_t *spins) {
    merge_body(N, R, n, amb, code, spins, blockIdx.x);
}

__global__ void k_merge_many(const MergeArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const MergeArgs a = as[k];
    merge_body(a.N, a.R, a.n, a.amb, a.code, a.spins, blockIdx.x);
}

hipError_t launch_merge(int N, int R, int n, const int32_t *amb, const int64_t *code,
                        int8_t *spins, hipStream_t st) {
    int64_t t = (int64_t)R * n;
    if (t == 0) return hipSuccess;
    k_merge<<<(unsigned)((t + 255) / 256), 256, 0, st>>>(N, R, n, amb, code, spins);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exact Ising energy (Eq. 1) and cut (Methods, MAX-CUT with w = J).
//
// Dense instances (k_energy_mv): with U = sum_{i<j} J_ij s_i s_j, S = sum_{i<j} J_ij and
// H = sum_i h_i s_i,  E = U + H  and  C = sum_{i<j, s_i != s_j} J_ij = (S - U) / 2.
// Every J is an integer m 2^b0 with |m| < 2^span; in D balanced base-256 digits d_k in
// [-128, 127] (span <= 8 D - 2), U's digit sums are products of int8 matrices: exact 32-bit
// integers y_k = d_k s per row (at most 256 N) and exact 64-bit ones Q_k = s y_k.  The
// merge adds the digit totals into the fixed-point accumulator and rounds once.
//
// CSR instances, and dense ones beyond D = 20 or near binary64's range (k_energy), keep
// one workgroup per (vector, slice): the sum over ordered pairs i != j counts each pair
// twice, so 2E = sum_{i!=j} J s s + 2 sum h s and 2C = sum_{i!=j, s_i != s_j} J are
// accumulated exactly (binary64 when the fast condition holds, else the fixed-point
// accumulator per term) and rounded with the scale halved.
// ---------------------------------------------------------------------------
struct EnArgs {
    int N, V, P, csr, b0;
    int fast;          // plain binary64 sums are exact (see launch_energy)
    const double *J;
    const int32_t *rp, *ci;
    const double *h;
    const int8_t *spins;
    void *part;        // [V][P] partials: two doubles (fast) or two Acc256
    double *E, *cut;
};

__device__ void block_acc_reduce(Acc256 &acc, Acc256 *sh) {
    acc_wave_allreduce(acc);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int v = 1; v < (int)(blockDim.x >> 6); v++) acc_merge(acc, sh[v]);
    __syncthreads();
}

// Sum of a binary64 value over the workgroup (exact when every partial sum is).
__device__ double block_sum(double x, double *sh) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = x;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int v = 0; v < (int)(blockDim.x >> 6); v++) t += sh[v];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(256) void k_energy(EnArgs a) {
    __shared__ Acc256 sh[4];
    __shared__ double shd[4];
    __shared__ int8_t sv[ENERGY_MAXN_LDS];
    const int v = blockIdx.x / a.P, p = blockIdx.x % a.P, tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int8_t *s = a.spins + (int64_t)v * a.N;
    const bool lds = a.N <= ENERGY_MAXN_LDS;
    if (lds)
        for (int i = tid; i < a.N; i += 256) sv[i] = s[i];
    __syncthreads();
    const int8_t *ss = lds ? sv : s;
    const int b0 = a.b0;
    const int64_t slot = (int64_t)v * a.P + p;
    if (a.fast) {
        // every partial sum is a multiple of 2^b0 below 2^(53 + b0): binary64 is exact
        double ae = 0.0, ac = 0.0;
        if (!a.csr) {
            for (int i = 4 * p + w; i < a.N; i += 4 * a.P) {
                const double *Jr = a.J + (int64_t)i * a.N;
                const int si = ss[i];
                for (int j = lane; j < a.N; j += 64) {
                    const double J = Jr[j];
                    const bool same = si == ss[j];
                    ae += same ? J : -J;
                    ac += same ? 0.0 : J;
                }
            }
        } else {
            for (int i = 256 * p + tid; i < a.N; i += 256 * a.P) {
                const int si = ss[i];
                for (int e = a.rp[i]; e < a.rp[i + 1]; e++) {
                    const double J = a.J[e];
                    const bool same = si == ss[a.ci[e]];
                    ae += same ? J : -J;
                    ac += same ? 0.0 : J;
                }
            }
        }
        for (int i = 256 * p + tid; i < a.N; i += 256 * a.P)
            ae += ss[i] > 0 ? 2.0 * a.h[i] : -2.0 * a.h[i];
        ae = block_sum(ae, shd);
        ac = block_sum(ac, shd);
        if (tid == 0) {
            double *o = (double *)a.part + 2 * slot;
            o[0] = ae;
            o[1] = ac;
        }
        return;
    }
    Acc256 ae, ac;
    acc_zero(ae);
    acc_zero(ac);
    if (!a.csr) {
        for (int i = 4 * p + w; i < a.N; i += 4 * a.P) {
            const double *Jr = a.J + (int64_t)i * a.N;
            const int si = ss[i];
            for (int j = lane; j < a.N; j += 64) {
                const double J = Jr[j];
                if (J == 0.0) continue;
                const int sj = ss[j];
                acc_add(ae, si == sj ? J : -J, b0);
                if (si != sj) acc_add(ac, J, b0);
            }
        }
    } else {
        for (int i = 256 * p + tid; i < a.N; i += 256 * a.P) {
            int si = ss[i];
            for (int e = a.rp[i]; e < a.rp[i + 1]; e++) {
                double J = a.J[e];
                int sj = ss[a.ci[e]];
                acc_add(ae, si == sj ? J : -J, b0);
                if (si != sj) acc_add(ac, J, b0);
            }
        }
    }
    for (int i = 256 * p + tid; i < a.N; i += 256 * a.P) {
        double hh = a.h[i];
        if (hh != 0.0) acc_add(ae, ss[i] > 0 ? 2.0 * hh : -2.0 * hh, b0);
    }
    block_acc_reduce(ae, sh);
    block_acc_reduce(ac, sh);
    if (tid == 0) {
        Acc256 *o = (Acc256 *)a.part + 2 * slot;
        o[0] = ae;
        o[1] = ac;
    }
}

// Totals of the P slices of each vector (a thread per vector), rounded once.
__global__ __launch_bounds__(64) void k_energy_merge(EnArgs a) {
    const int v = blockIdx.x * 64 + threadIdx.x;
    if (v >= a.V) return;
    const int64_t s0 = (int64_t)v * a.P;
    if (a.fast) {
        const double *o = (const double *)a.part;
        double ae = 0.0, ac = 0.0;
        for (int p = 0; p < a.P; p++) {
            ae += o[2 * (s0 + p)];
            ac += o[2 * (s0 + p) + 1];
        }
        if (a.E) a.E[v] = 0.5 * ae;
        if (a.cut) a.cut[v] = 0.5 * ac;
        return;
    }
    const Acc256 *o = (const Acc256 *)a.part;
    Acc256 ae = o[2 * s0], ac = o[2 * s0 + 1];
    for (int p = 1; p < a.P; p++) {
        acc_merge(ae, o[2 * (s0 + p)]);
        acc_merge(ac, o[2 * (s0 + p) + 1]);
    }
    if (a.E) a.E[v] = acc_round(ae, a.b0 - 1);
    if (a.cut) a.cut[v] = acc_round(ac, a.b0 - 1);
}

// ----- dense: many vectors per pass, digit sums -----
struct EnMvArgs {
    int N, V, P, b0;
    int jt;            // type of Js (JT_F32, JT_BF16, JT_FP8), -1 to read J
    int ldj;           // row pitch of Js
    const void *Js;    // the exact storage copy of J (or NULL)
    const double *J;
    const double *h;   // null without fields
    const int8_t *spins;
    int64_t *part;     // [P][V][D] Q = 2 U, then [P][D] S2 = 2 S
    double scale;      // 2^-b0
    double *E, *cut;
};

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4_r;

// Balanced digits of 16 couplings, by digit: A[k] holds the digits k (one MFMA operand of a
// lane).  m = x 2^-b0 is split into 32-bit words from the top: adding 2^52 rounds to an integer
// and leaves it in the low word, fma takes it off exactly.  With 0x80808080 added as well the
// word's bytes are d_k + 128, and bit 32 is the carry into the next word.
template <int D>
__device__ __forceinline__ void mv_digits(const double (&x)[16], double scale, i32x4_r (&A)[D]) {
    constexpr int NWD = (D + 3) / 4;
    constexpr double LOW = 0x1p52 + 2155905152.0, TOP = 0x1.8p52 + 2155905152.0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        uint32_t wd[4][NWD];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const double v = x[4 * q + e];
            if constexpr (NWD == 1) {
                wd[e][0] = (uint32_t)__double_as_longlong(__builtin_fma(v, scale, TOP)) ^ 0x80808080u;
            } else {
                double rem = v * scale, p32 = 1.0;
#pragma unroll
                for (int w = 1; w < NWD; w++) p32 *= 0x1p32;
                uint32_t hi[NWD];
#pragma unroll
                for (int w = NWD - 1; w >= 0; w--, p32 *= 0x1p-32) {
                    const double m = w == NWD - 1 ? TOP : LOW;
                    const double t = __builtin_fma(rem, 1.0 / p32, m);
                    if (w) rem = __builtin_fma(t - m, -p32, rem);
                    const uint64_t b = (uint64_t)__double_as_longlong(t);
                    wd[e][w] = (uint32_t)b;
                    hi[w] = (uint32_t)(b >> 32) & 1u;
                }
                uint32_t carry = hi[0];
#pragma unroll
                for (int w = 1; w < NWD; w++) {
                    const uint32_t t = wd[e][w] + carry;
                    if (w + 1 < NWD) carry = hi[w] | (uint32_t)(t < carry);
                    wd[e][w] = t;
                }
#pragma unroll
                for (int w = 0; w < NWD; w++) wd[e][w] ^= 0x80808080u;
            }
        }
#pragma unroll
        for (int w = 0; w < NWD; w++) {                  // 4 x 4 byte transposes
            const uint32_t a01 = __builtin_amdgcn_perm(wd[1][w], wd[0][w], 0x05010400u);
            const uint32_t a23 = __builtin_amdgcn_perm(wd[3][w], wd[2][w], 0x05010400u);
            if (4 * w < D) A[4 * w][q] = (int)__builtin_amdgcn_perm(a23, a01, 0x05040100u);
            if (4 * w + 1 < D) A[4 * w + 1][q] = (int)__builtin_amdgcn_perm(a23, a01, 0x07060302u);
            const uint32_t b01 = __builtin_amdgcn_perm(wd[1][w], wd[0][w], 0x07030602u);
            const uint32_t b23 = __builtin_amdgcn_perm(wd[3][w], wd[2][w], 0x07030602u);
            if (4 * w + 2 < D) A[4 * w + 2][q] = (int)__builtin_amdgcn_perm(b23, b01, 0x05040100u);
            if (4 * w + 3 < D) A[4 * w + 3][q] = (int)__builtin_amdgcn_perm(b23, b01, 0x07060302u);
        }
    }
}

// Couplings of a row in a block of 64 columns from 64 c, zeros past the last column.  A storage
// copy gives lane group kg the columns 16 kg .. + 15; binary64 couplings go out in pieces of
// two, columns 8 j + 2 kg, + 1 (j = 0 .. 7), so that a load of the four groups is 64
// consecutive bytes instead of pieces 128 bytes apart.
__device__ __forceinline__ void mv_load(const EnMvArgs &a, int row, int c, int kg, double (&x)[16]) {
    typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
    if (a.jt >= 0) {                                     // padded with zeros, pieces aligned
        const int64_t t = (int64_t)row * a.ldj + min(64 * c + 16 * kg, (a.N - 1) & ~15);
        if (a.jt == JT_FP8) {
            const i32x4_r w = *(const i32x4_r *)((const uint8_t *)a.Js + t);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                x[4 * q] = __builtin_amdgcn_cvt_f32_fp8(w[q], 0);
                x[4 * q + 1] = __builtin_amdgcn_cvt_f32_fp8(w[q], 1);
                x[4 * q + 2] = __builtin_amdgcn_cvt_f32_fp8(w[q], 2);
                x[4 * q + 3] = __builtin_amdgcn_cvt_f32_fp8(w[q], 3);
            }
        } else if (a.jt == JT_BF16) {
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const i32x4_r w = *(const i32x4_r *)((const uint16_t *)a.Js + t + 8 * q);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    x[8 * q + 2 * e] = __uint_as_float((uint32_t)w[e] << 16);
                    x[8 * q + 2 * e + 1] = __uint_as_float((uint32_t)w[e] & 0xffff0000u);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const float4 f = *(const float4 *)((const float *)a.Js + t + 4 * q);
                x[4 * q] = f.x; x[4 * q + 1] = f.y; x[4 * q + 2] = f.z; x[4 * q + 3] = f.w;
            }
        }
        return;
    }
    const int k = 64 * c + 2 * kg;
    const double *Jr = a.J + (int64_t)row * a.N + k;
    if (64 * c + 64 <= a.N) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const d2 d = *(const d2 *)(Jr + 8 * j);
            x[2 * j] = d[0];
            x[2 * j + 1] = d[1];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int o = 8 * (e >> 1) + (e & 1);
            x[e] = k + o < a.N ? Jr[o] : 0.0;
        }
    }
}

// 16 consecutive spins of a vector from column k < N, a multiple of 16 (columns past the end:
// any value).
__device__ __forceinline__ i32x4_r mv_spins(const EnMvArgs &a, int v, int k) {
    typedef i32x4_r i4u __attribute__((aligned(1)));
    const int8_t *s = a.spins + (int64_t)v * a.N + k;
    i32x4_r x = {0, 0, 0, 0};
    if (k + 16 <= a.N) {
        x = *(const i4u *)s;
    } else {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            uint32_t w = 0;
#pragma unroll
            for (int e = 0; e < 4; e++)
                w |= k + 4 * q + e < a.N ? (uint32_t)(uint8_t)s[4 * q + e] << (8 * e) : 0u;
            x[q] = (int)w;
        }
    }
    return x;
}

// Bytes +-1 by the sign bits.
__device__ __forceinline__ i32x4_r mv_signs(i32x4_r x) {
#pragma unroll
    for (int q = 0; q < 4; q++)
        x[q] = (int)((((uint32_t)x[q] >> 7) & 0x01010101u) * 0xfeu ^ 0x01010101u);
    return x;
}

// Spins of columns 16 kg .. + 15 by lane group to the order of the binary64 couplings: word q
// of group kg becomes columns 16 q + 2 kg, + 1, + 8 + 2 kg, + 9 + 2 kg.  The words for each
// group within a lane, then a 4 x 4 transpose over the lane groups.
__device__ __forceinline__ i32x4_r mv_order(i32x4_r x) {
    uint32_t w0 = __builtin_amdgcn_perm(x[2], x[0], 0x05040100u);
    uint32_t w1 = __builtin_amdgcn_perm(x[2], x[0], 0x07060302u);
    uint32_t w2 = __builtin_amdgcn_perm(x[3], x[1], 0x05040100u);
    uint32_t w3 = __builtin_amdgcn_perm(x[3], x[1], 0x07060302u);
    const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    return (i32x4_r){(int)c[0], (int)c[1], (int)d[0], (int)d[1]};
}

// A wavefront takes VEC vectors and a contiguous range of the blocks of 16 rows x 64 columns
// that reach the diagonal or lie above it, in row order, the next block's couplings in flight.
// A 16-column tile has weight 0 below the diagonal, 1 on it and 2 above: with it Q = sum over
// ordered pairs = 2 U.  The weight goes to the spins, D 16x16x64 int8 MFMAs per 16 vectors do
// the rest, and at the end of a block row y is folded into Q.  Bound by vector instructions:
// the digits (about 14 a coupling), the spins' order and the folds, which is why a wavefront
// takes as many vectors as its accumulators allow.  Measured at N = 5000, V = 256 real
// couplings (D = 7): 1040 us as masked binary64 multiply-adds on exact parts of J, 440 us as
// binary64 MFMAs on those, 170 us this way (211 us with 32 vectors a wavefront; 233 us with
// digits shifted out of the significand and 16 consecutive couplings a lane); 8 instances of
// N = 2000, V = 64, FP8 couplings (D = 1): 639 us, now 103 us.
template <int VEC, int D>
__device__ __forceinline__ void energy_mv_body(const EnMvArgs &a, const int bx_, const int by_) {
    constexpr int NT = VEC / 16;
    __shared__ int64_t red[4][VEC][D], reds[4][D];
    const int tid = threadIdx.x, lane = tid & 63, kg = lane >> 4, l16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = bx_, v0 = by_ * VEC;
    const bool first = by_ == 0;
    const int klast = (a.N - 1) & ~15;
    const int nt = (a.N + 15) / 16, nc = (a.N + 63) / 64;
    // blocks of row I: columns I / 4 .. nc - 1; rows 4 B .. 4 B + 3 start at B (4 nc - 2 (B - 1))
    auto start = [&](int r) {
        const int64_t B = r >> 2;
        return B * (4ll * nc - 2 * (B - 1)) + (int64_t)(r & 3) * (nc - B);
    };
    // this wavefront's share: a row's fold counts as a block, so short rows are not the slowest
    const int64_t nw = 4ll * a.P, g = 4 * p + w;
    auto locate = [&](int64_t x, int &row) {             // first block at or after cost x
        int lo = 0, hi = nt - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (start(mid) + mid <= x) lo = mid;
            else hi = mid - 1;
        }
        row = lo;
        const int64_t off = x - start(lo) - lo - 1;
        return start(lo) + (off > 0 ? off : 0);
    };
    const int64_t cost = start(nt) + nt;
    int I, Ie;
    const int64_t u1 = locate(cost * (g + 1) / nw, Ie);
    int64_t u = locate(cost * g / nw, I);
    int c = (I >> 2) + (int)(u - start(I));
    const int vl = v0 + l16;

    int64_t q[NT][D], s2[D];
    i32x4_r y[NT][D];
    int s2i[D];
#pragma unroll
    for (int k = 0; k < D; k++) {
        s2[k] = 0;
        s2i[k] = 0;
#pragma unroll
        for (int t = 0; t < NT; t++) {
            q[t][k] = 0;
            y[t][k] = (i32x4_r){0, 0, 0, 0};
        }
    }
    const bool nat = a.jt >= 0;                          // couplings in column order
    double x[16];
    i32x4_r raw[NT];
    if (u < u1) {
        mv_load(a, min(16 * I + l16, a.N - 1), c, kg, x);
#pragma unroll
        for (int n = 0; n < NT; n++)
            raw[n] = mv_spins(a, min(vl + 16 * n, a.V - 1), min(64 * c + 16 * kg, klast));
    }
    for (; u < u1; u++) {
        i32x4_r A[D];
        mv_digits<D>(x, a.scale, A);
        const int In = c + 1 < nc ? I : I + 1, cn = c + 1 < nc ? c + 1 : (I + 1) >> 2;
        if (u + 1 < u1) mv_load(a, min(16 * In + l16, a.N - 1), cn, kg, x);
        // weights 0, 1, 2 of this lane's words: the shift and the mask of their spins
        int wgt[4];
        uint32_t keep[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int ct = 4 * c + (nat ? kg : q);       // the word's 16-column tile
            wgt[q] = ct < I || 16 * ct >= a.N ? 0 : ct == I ? 1 : 2;
            keep[q] = wgt[q] == 0 ? 0u : wgt[q] == 1 ? 0xffffffffu : 0xfefefefeu;
        }
        if (first) {
            const bool in = 16 * I + l16 < a.N;
#pragma unroll
            for (int k = 0; k < D; k++)
#pragma unroll
                for (int q = 0; q < 4; q++)
                    s2i[k] += in ? wgt[q] * __builtin_amdgcn_sdot4(A[k][q], 0x01010101, 0, false) : 0;
        }
#pragma unroll
        for (int n = 0; n < NT; n++) {
            i32x4_r sp = mv_signs(raw[n]);
            if (!nat) sp = mv_order(sp);
            if (u + 1 < u1)
                raw[n] = mv_spins(a, min(vl + 16 * n, a.V - 1), min(64 * cn + 16 * kg, klast));
#pragma unroll
            for (int q = 0; q < 4; q++)                  // doubled: 0x01 -> 0x02, 0xff -> 0xfe
                sp[q] = (int)(((uint32_t)sp[q] << (wgt[q] >> 1)) & keep[q]);
#pragma unroll
            for (int k = 0; k < D; k++)
                y[n][k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[k], sp, y[n][k], 0, 0, 0);
        }
        if (In != I || u + 1 == u1) {
            // Q += s_i y_i: accumulator v of a lane is row 16 I + 4 kg + v, vector l16; the four
            // rows stay below 1024 N <= 2^30
            const int i0 = 16 * I + 4 * kg;
            const bool full = 16 * I + 16 <= a.N;
#pragma unroll
            for (int n = 0; n < NT; n++) {
                const int8_t *sr = a.spins + (int64_t)min(vl + 16 * n, a.V - 1) * a.N;
                int m[4], ms = 0;                        // -1 where the spin is -1
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    m[v] = (int)sr[min(i0 + v, a.N - 1)] >> 31;
                    ms -= m[v];
                }
                if (!full) {
                    ms = 0;
#pragma unroll
                    for (int v = 0; v < 4; v++) {
                        ms -= i0 + v < a.N ? m[v] : 0;
#pragma unroll
                        for (int k = 0; k < D; k++) y[n][k][v] = i0 + v < a.N ? y[n][k][v] : 0;
                        m[v] = i0 + v < a.N ? m[v] : 0;
                    }
                }
#pragma unroll
                for (int k = 0; k < D; k++) {
                    const int t = (y[n][k][0] ^ m[0]) + ((y[n][k][1] ^ m[1]) + ((y[n][k][2] ^ m[2]) +
                                  ((y[n][k][3] ^ m[3]) + ms)));
                    q[n][k] += (int64_t)t;
                    y[n][k] = (i32x4_r){0, 0, 0, 0};
                }
            }
#pragma unroll
            for (int k = 0; k < D; k++) {
                s2[k] += s2i[k];
                s2i[k] = 0;
            }
        }
        I = In;
        c = cn;
    }
#pragma unroll
    for (int n = 0; n < NT; n++)
#pragma unroll
        for (int k = 0; k < D; k++) {
            int64_t t = q[n][k];
            t += (int64_t)__shfl_xor((long long)t, 16);
            t += (int64_t)__shfl_xor((long long)t, 32);
            if (kg == 0) red[w][16 * n + l16][k] = t;
        }
#pragma unroll
    for (int k = 0; k < D; k++) {
        int64_t t = s2[k];
        for (int o = 32; o > 0; o >>= 1) t += (int64_t)__shfl_xor((long long)t, o);
        if (lane == 0) reds[w][k] = t;
    }
    __syncthreads();
    for (int e = tid; e < VEC * D; e += 256) {
        const int v = e / D, k = e % D;
        if (v0 + v < a.V)
            a.part[((int64_t)p * a.V + v0 + v) * D + k] =
                red[0][v][k] + red[1][v][k] + red[2][v][k] + red[3][v][k];
    }
    if (first && tid < D)
        a.part[(int64_t)a.P * a.V * D + (int64_t)p * D + tid] =
            reds[0][tid] + reds[1][tid] + reds[2][tid] + reds[3][tid];
}

template <int VEC, int D>
__global__ __launch_bounds__(256) void k_energy_mv(EnMvArgs a) {
    energy_mv_body<VEC, D>(a, blockIdx.x, blockIdx.y);
}

// Many instances: instance blockIdx.z, its own slice count nb[z] (= its a.P).
template <int VEC, int D>
__global__ __launch_bounds__(256) void k_energy_mv_many(const EnMvArgs *as, const int *nb) {
    const int k = blockIdx.z;
    if ((int)blockIdx.x >= nb[k]) return;
    const EnMvArgs a = as[k];
    energy_mv_body<VEC, D>(a, blockIdx.x, blockIdx.y);
}

// Per vector (one wavefront): digit totals over the slices and of H = sum h_i s_i (h shares J's
// digits), then E = (Q + 2 H) / 2 and C = (S2 - Q) / 4, each rounded once.  The slices of a digit
// are added as integers, so that only the D lanes of the digits meet in the accumulators.  Bound
// by their shuffles where the vectors are many and the spins few (N = 64, V = 100,000: D = 1 278 us
// with all 64 lanes in the accumulators, 111 now; D = 10 332 and 203).
template <int D>
__device__ __forceinline__ void energy_mv_merge_body(const EnMvArgs &a, const int bx_) {
    const int v = bx_ * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (v >= a.V) return;
    constexpr int G = 64 / D;
    constexpr int NP = D > 16 ? 32 : D > 8 ? 16 : D > 4 ? 8 : D;   // lanes of the digits, a power of two
    const int k = lane % D, p0 = lane / D;               // slices p0, p0 + G, ...
    int64_t Q = 0, S = 0;
    if (p0 < G)
#pragma unroll 4
        for (int p = p0; p < a.P; p += G) {
            Q += a.part[((int64_t)p * a.V + v) * D + k];
            S += a.part[(int64_t)a.P * a.V * D + (int64_t)p * D + k];
        }
    if (a.P > 1) {                                       // lane k < D: the sum over lanes k, k + D, ...
        int64_t q = Q, s = S;
        for (int g = 1; g < min(G, a.P); g++) {
            q += (int64_t)__shfl((long long)Q, k + D * g);
            s += (int64_t)__shfl((long long)S, k + D * g);
        }
        Q = q;
        S = s;
    }
    int64_t T = Q;                                       // Q + 2 H by digit
    if (a.h) {
        int hs[D], o0 = 32;
        while (o0 && 16 * o0 >= a.N) o0 >>= 1;            // the lanes 2 o0 .. 63 hold no spin
#pragma unroll
        for (int d = 0; d < D; d++) hs[d] = 0;
        for (int i = 16 * lane; i < a.N; i += 1024) {
            double x[16];
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = i + e < a.N ? a.h[i + e] : 0.0;
            i32x4_r A[D];
            mv_digits<D>(x, a.scale, A);
            const i32x4_r sp = mv_signs(mv_spins(a, v, i));
#pragma unroll
            for (int d = 0; d < D; d++)
#pragma unroll
                for (int q = 0; q < 4; q++) hs[d] = __builtin_amdgcn_sdot4(A[d][q], sp[q], hs[d], false);
        }
#pragma unroll
        for (int d = 0; d < D; d++) {
            int t = hs[d];
            for (int o = o0; o > 0; o >>= 1) t += __shfl_xor(t, o);
            t = __builtin_amdgcn_readfirstlane(t);
            if (lane == d) T += 2 * (int64_t)t;
        }
    }
    Acc256 ae, ac;
    acc_zero(ae);
    acc_zero(ac);
    if (lane < D) {
        // |Q_k|, |S_k| <= 128 N^2, together below 2^53
        acc_add(ae, ldexp((double)T, a.b0 + 8 * k), a.b0);
        acc_add(ac, ldexp((double)(S - Q), a.b0 + 8 * k), a.b0);
    }
    acc_wave_allreduce<NP>(ae);
    acc_wave_allreduce<NP>(ac);
    if (lane) return;
    if (a.E) a.E[v] = acc_round(ae, a.b0 - 1);
    if (a.cut) a.cut[v] = acc_round(ac, a.b0 - 2);
}

template <int D>
__global__ __launch_bounds__(256) void k_energy_mv_merge(EnMvArgs a) {
    energy_mv_merge_body<D>(a, blockIdx.x);
}

template <int D>
__global__ __launch_bounds__(256) void k_energy_mv_merge_many(const EnMvArgs *as, const int *nb) {
    const int k = blockIdx.y;
    if ((int)blockIdx.x >= nb[k]) return;
    const EnMvArgs a = as[k];
    energy_mv_merge_body<D>(a, blockIdx.x);
}

// Digits of the many-vector kernel for instance I (0: it does not apply): the smallest count it
// is built for with 8 D - 2 >= span; every digit total has to stay a normal binary64 number.
static int energy_digits(const Instance &I) {
    if (I.layout != HQA_DENSE || I.es.lsb == INT32_MIN) return 0;
    const int span = I.es.msb + 1 - I.es.lsb;
    if (I.es.msb > 900 || I.es.lsb < -900 || I.N > (1 << 20)) return 0;
    for (int k = 0; k < MV_NDIGITS; k++)
        if (8 * MV_DIGITS[k] - 2 >= span) return MV_DIGITS[k];
    return 0;
}

static EnMvArgs energy_mv_args(const Instance &I, int V, int P, const int8_t *spins, double *E,
                               double *cut, void *part) {
    EnMvArgs m;
    m.N = I.N; m.V = V; m.b0 = I.es.lsb; m.P = P;
    m.J = I.J64; m.h = I.has_h ? I.h64 : nullptr; m.spins = spins; m.E = E; m.cut = cut;
    // the compact storage copy when it holds every coupling exactly
    m.jt = -1; m.ldj = 0; m.Js = nullptr;
    if (I.js_exact && I.Js) {
        m.jt = (int)I.jt; m.ldj = I.Np; m.Js = I.Js;
    }
    m.part = (int64_t *)part;
    m.scale = std::ldexp(1.0, -I.es.lsb);
    return m;
}

// k_energy_mv or its batched form for (vec, D): f(integral constants) over the built pairs.
template <class F>
static void energy_mv_dispatch(int vec, int D, F f) {
#define HQA_MV(VV, DD) if (vec == VV && D == DD) f(std::integral_constant<int, VV>(), std::integral_constant<int, DD>());
    HQA_MV(16, 1) HQA_MV(16, 2) HQA_MV(16, 4) HQA_MV(16, 7) HQA_MV(16, 8) HQA_MV(16, 10)
    HQA_MV(16, 12) HQA_MV(16, 16) HQA_MV(16, 20) HQA_MV(32, 10) HQA_MV(32, 12)
    HQA_MV(64, 1) HQA_MV(64, 2) HQA_MV(64, 4) HQA_MV(64, 7) HQA_MV(64, 8)
#undef HQA_MV
}

hipError_t launch_energy(const Instance &I, int V, const int8_t *spins, double *E, double *cut,
                         void *part, hipStream_t st) {
    if (V == 0) return hipSuccess;
    const int D = energy_by_vector(I.N, V) ? 0 : energy_digits(I);
    if (D) {
        const EnergyPlan pl = energy_plan(I.N, V, D);
        for (int v0 = 0; v0 < V; v0 += pl.piece) {
            const int n = std::min(pl.piece, V - v0);
            const EnMvArgs m = energy_mv_args(I, n, pl.P, spins + (int64_t)v0 * I.N, E ? E + v0 : nullptr,
                                              cut ? cut + v0 : nullptr, part);
            energy_mv_dispatch(pl.vec, D, [&](auto vv, auto dd) {
                k_energy_mv<vv.value, dd.value><<<dim3(m.P, (n + pl.vec - 1) / pl.vec), 256, 0, st>>>(m);
                k_energy_mv_merge<dd.value><<<(n + 3) / 4, 256, 0, st>>>(m);
            });
        }
        return hipGetLastError();
    }
    EnArgs a;
    a.N = I.N; a.V = V; a.P = energy_slices(I.N, V); a.csr = I.layout == HQA_CSR; a.b0 = I.es.lsb;
    // Every J and h is a multiple of 2^lsb below 2^(msb + 1); the sums take at most
    // N^2 + N terms of magnitude below 2^(msb + 2) (2h).  When those fit 53 bits above
    // 2^lsb, every partial binary64 sum is exact, whatever the order.
    {
        const double terms = (double)I.N * I.N + I.N;
        int lg = 0;
        while (lg < 64 && std::ldexp(1.0, lg) < terms) lg++;
        a.fast = I.es.lsb != INT32_MIN && (I.es.msb + 2 - I.es.lsb) + lg <= 52;
    }
    a.J = I.J64; a.rp = I.rp; a.ci = I.ci; a.h = I.h64; a.spins = spins; a.part = part;
    a.E = E; a.cut = cut;
    k_energy<<<V * a.P, 256, 0, st>>>(a);
    k_energy_merge<<<(V + 63) / 64, 64, 0, st>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The read-out of many instances (same R, n and solve) in one launch per stage: every
// stage's kernel runs for all instances at once (instance = the last grid dimension,
// each with its own block count), in the order select, reduce, enumerate, merge,
// energy, so the many small grids of one instance no longer leave the device idle.
// Each stage computes exactly what the per-instance launches compute.
// ---------------------------------------------------------------------------
namespace {
struct Blob {
    std::vector<uint8_t> h;
    size_t put(const void *p, size_t n) {
        const size_t off = (h.size() + 255) & ~(size_t)255;
        h.resize(off + n);
        memcpy(h.data() + off, p, n);
        return off;
    }
};
template <class T>
size_t put_vec(Blob &b, const std::vector<T> &v) { return b.put(v.data(), v.size() * sizeof(T)); }
}  // namespace

size_t readout_batch_arg_bytes(int count) {
    // the argument arrays and their block counts, each rounded to 256 bytes
    const size_t per = sizeof(EnMvArgs) + sizeof(EnumRealArgs) + sizeof(EnumArgs) + sizeof(SelArgs) +
                       sizeof(RedArgs) + sizeof(MergeArgs) + 24 * sizeof(int);
    return (size_t)count * per + 40 * 256;
}

hipError_t launch_readout_batch(const std::vector<ReadoutJob> &jobs, int R, int n, int solve,
                                void *argbuf, size_t argcap, hipStream_t st, int mode) {
    const int count = (int)jobs.size();
    if (count == 0) return hipSuccess;
    Blob b;
    // select
    std::vector<SelArgs> sel(count);
    std::vector<int> nsel(count, R);
    for (int c = 0; c < count; c++) {
        const ReadoutJob &j = jobs[c];
        SelArgs &a = sel[c];
        a.N = j.I->N; a.R = R; a.ld = j.I->ld; a.smaj = j.I->smaj; a.f64 = j.prec == HQA_PREC_F64_REF;
        a.W = j.W; a.n = n; a.S64 = j.I->S64; a.S32 = j.I->S32; a.amb = j.amb; a.spins = j.spins;
        a.keys = nullptr;
    }
    const size_t o_sel = put_vec(b, sel), o_nsel = put_vec(b, nsel);
    // reduce, enumerate, merge (exact solution of the reduced problems)
    const bool solving = solve && n > 0;
    std::vector<RedArgs> red;
    std::vector<EnumRealArgs> er;
    std::vector<EnumArgs> ei;
    std::vector<MergeArgs> mg;
    std::vector<int> nred, ner, nmid, nei, nmg;
    const int pt = n < ENUM_PT_REAL ? n : ENUM_PT_REAL;
    const int Pe = ((1 << pt) + 255) / 256;
    if (solving) {
        for (int c = 0; c < count; c++) {
            const ReadoutJob &j = jobs[c];
            const Instance &I = *j.I;
            RedArgs a;
            a.N = I.N; a.R = R; a.n = n; a.csr = I.layout == HQA_CSR; a.b0 = I.es.lsb;
            a.words = reduce_words(I, n);
            a.scale = a.words ? std::ldexp(1.0, -I.es.lsb) : 0.0;
            a.J = I.J64; a.rp = I.rp; a.ci = I.ci; a.h = I.h64;
            a.amb = j.amb; a.spins = j.spins; a.h_eff = j.h_eff; a.J_eff = j.J_eff;
            red.push_back(a);
            nred.push_back((R * n + 3) / 4);
            if (!I.j_integral) {
                EnumRealArgs e;
                e.n = n; e.R = R; e.P = Pe; e.b0 = I.es.lsb;
                e.J_eff = j.J_eff; e.h_eff = j.h_eff; e.code = j.code; e.e_red = j.e_red;
                e.partE = (double *)j.escr;
                e.partC = (int64_t *)((char *)j.escr + (size_t)R * e.P * 8);
                e.thresh = (double *)((char *)j.escr + (size_t)R * e.P * 16);
                er.push_back(e);
                ner.push_back(R * Pe);
                nmid.push_back(R);
            } else {
                EnumArgs e;
                e.n = n; e.R = R; e.b0 = I.es.lsb; e.integral = 1;
                e.J_eff = j.J_eff; e.h_eff = j.h_eff; e.code = j.code; e.e_red = j.e_red;
                ei.push_back(e);
                nei.push_back(R);
            }
            MergeArgs m;
            m.N = I.N; m.R = R; m.n = n; m.amb = j.amb; m.code = j.code; m.spins = j.spins;
            mg.push_back(m);
            nmg.push_back((R * n + 255) / 256);
        }
    }
    const size_t o_red = put_vec(b, red), o_nred = put_vec(b, nred);
    const size_t o_er = put_vec(b, er), o_ner = put_vec(b, ner), o_nmid = put_vec(b, nmid);
    const size_t o_ei = put_vec(b, ei), o_nei = put_vec(b, nei);
    const size_t o_mg = put_vec(b, mg), o_nmg = put_vec(b, nmg);
    // energy: the many-vector kernel by digit count; others one instance at a time
    std::vector<EnMvArgs> mv[MV_NDIGITS];
    std::vector<int> nmv[MV_NDIGITS], nmm[MV_NDIGITS];   // slices of the sums, blocks of the merge
    std::vector<int> fallback;
    for (int c = 0; c < count; c++) {
        const ReadoutJob &j = jobs[c];
        const int D = energy_digits(*j.I);
        const EnergyPlan pl = D ? energy_plan(j.I->N, R, D) : EnergyPlan{0, 0, 0};
        if (!D || pl.piece < R) {
            fallback.push_back(c);
            continue;
        }
        const int x = (int)(std::find(MV_DIGITS, MV_DIGITS + MV_NDIGITS, D) - MV_DIGITS);
        mv[x].push_back(energy_mv_args(*j.I, R, pl.P, j.spins, j.E, j.C, j.part));
        nmv[x].push_back(mv[x].back().P);
        nmm[x].push_back((R + 3) / 4);
    }
    size_t o_mv[MV_NDIGITS] = {}, o_nmv[MV_NDIGITS] = {}, o_nmm[MV_NDIGITS] = {};
    for (int x = 0; x < MV_NDIGITS; x++) {
        o_mv[x] = put_vec(b, mv[x]);
        o_nmv[x] = put_vec(b, nmv[x]);
        o_nmm[x] = put_vec(b, nmm[x]);
    }
    if (b.h.size() > argcap) return hipErrorInvalidValue;
    // the host copy of the arguments lives only in this call: wait for the upload
    hipError_t e = hipSuccess;
    if (mode != READOUT_LAUNCH) {
        e = hipMemcpyAsync(argbuf, b.h.data(), b.h.size(), hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess || mode == READOUT_UPLOAD) return e;
    }
    uint8_t *d = (uint8_t *)argbuf;
    auto mx = [](const std::vector<int> &v) { int m = 0; for (int x : v) m = std::max(m, x); return m; };
    k_select_many<<<dim3(R, count), 256, 0, st>>>((const SelArgs *)(d + o_sel), (const int *)(d + o_nsel));
    if (solving) {
        k_reduce_many<<<dim3(mx(nred), count), 256, 0, st>>>((const RedArgs *)(d + o_red),
                                                            (const int *)(d + o_nred));
        if (!er.empty()) {
            const EnumRealArgs *as = (const EnumRealArgs *)(d + o_er);
            const int *nr = (const int *)(d + o_ner), *nm = (const int *)(d + o_nmid);
            const int ce = (int)er.size();
            for (int pass = 1; pass <= 2; pass++) {
                switch (n - pt) {
#define HQA_ER(NL) case NL: if (pass == 1) k_enum_real_many<NL, 1><<<dim3(R * Pe, ce), 256, 0, st>>>(as, nr); \
                    else k_enum_real_many<NL, 2><<<dim3(R * Pe, ce), 256, 0, st>>>(as, nr); break;
                    HQA_ER(0) HQA_ER(1) HQA_ER(2) HQA_ER(3) HQA_ER(4) HQA_ER(5) HQA_ER(6)
                    HQA_ER(7) HQA_ER(8) HQA_ER(9) HQA_ER(10) HQA_ER(11)
                    HQA_ER(12)
#undef HQA_ER
                }
                k_enum_real_mid_many<<<dim3(R, ce), 64, 0, st>>>(as, nm, pass);
            }
        }
        if (!ei.empty()) {
            const EnumArgs *as = (const EnumArgs *)(d + o_ei);
            const int *ni = (const int *)(d + o_nei);
            const int ci = (int)ei.size();
            switch (n > ENUM_PT ? n - ENUM_PT : 0) {
#define HQA_EI(NL) case NL: k_enumerate_int_many<NL><<<dim3(R, ci), 1024, 0, st>>>(as, ni); break;
                HQA_EI(0) HQA_EI(1) HQA_EI(2) HQA_EI(3) HQA_EI(4) HQA_EI(5) HQA_EI(6) HQA_EI(7)
                HQA_EI(8) HQA_EI(9) HQA_EI(10) HQA_EI(11) HQA_EI(12) HQA_EI(13)
                default: k_enumerate_int_many<14><<<dim3(R, ci), 1024, 0, st>>>(as, ni); break;
#undef HQA_EI
            }
        }
        k_merge_many<<<dim3(mx(nmg), count), 256, 0, st>>>((const MergeArgs *)(d + o_mg),
                                                          (const int *)(d + o_nmg));
    }
    for (int x = 0; x < MV_NDIGITS; x++) {
        if (mv[x].empty()) continue;
        const int D = MV_DIGITS[x], vec = energy_mv_vec(R, D), cl = (int)mv[x].size();
        const EnMvArgs *as = (const EnMvArgs *)(d + o_mv[x]);
        const int *np = (const int *)(d + o_nmv[x]), *nq = (const int *)(d + o_nmm[x]);
        energy_mv_dispatch(vec, D, [&](auto vv, auto dd) {
            k_energy_mv_many<vv.value, dd.value>
                <<<dim3(mx(nmv[x]), (R + vec - 1) / vec, cl), 256, 0, st>>>(as, np);
            k_energy_mv_merge_many<dd.value><<<dim3((R + 3) / 4, cl), 256, 0, st>>>(as, nq);
        });
    }
    for (int c : fallback) {
        const ReadoutJob &j = jobs[c];
        e = launch_energy(*j.I, R, j.spins, j.E, j.C, j.part, st);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Single-flip tabu search on each replica's reduced problem, for n beyond exact
// enumeration (the paper hands n = 1000 ambivalent spins to a tabu search in its
// K2000 experiment; the search itself is this library's reading):
//   x = the read-out of the ambivalent spins; f_a = h_eff_a + sum_{b != a} J_ab x_b
//   (b ascending); D = 0, D_best = 0; for t = 1 .. iters: d_a = -2 x_a f_a; a move is
//   allowed when tabu_until[a] < t or D + d_a < D_best; a* = the allowed a with the
//   smallest d_a (ties: smallest a); D += d_a*; f_b -= 2 J_a*b x_a* (old value) for
//   b != a*; x_a* = -x_a*; tabu_until[a*] = t + tenure; if D < D_best keep x.
// One workgroup per replica.  A move is a chain of dependent latencies: the best candidate of
// each thread, wavefront and workgroup, then one load of the chosen row's couplings, so the
// search runs in few wavefronts with several spins a thread (one barrier per move, candidate
// slots double-buffered by parity), and
//  * k_tabu_int, for integral couplings and fields with small sums, keeps 2^13 d_a + (2 a +
//    [x_a > 0]) in one signed 32-bit word, whose order is that of (gain, index), so that a
//    reduction level is one minimum; J comes from the instance's compact exact copy where it
//    has one (1 to 4 bytes a coupling: an L2's worth instead of the memory-side cache);
//  * k_tabu, for real couplings, takes the minimum of the gains first and settles ties by
//    index only among lanes that hold it.
// The operations are those of the definition in binary64 without contraction (integers of
// that size are exact in both), so the trajectory is the same whatever the launch shape.
// Measured per move: K2000, R = 16, n = 1000: 1024 threads, candidates (gain, index) reduced as
// pairs and binary64 couplings 1.66 us; k_tabu_int 0.67 us (256, 1024
// threads 0.87, 0.85). Real couplings, N = 2000, n = 1000: 1.64 -> 1.13 us; n = 60: 1.37 -> 0.37 (0.26
// integral).
// ---------------------------------------------------------------------------
struct TabuArgs {
    int N, R, n, csr, tenure;
    int64_t iters;
    const double *J;
    const void *Js;       // compact exact copy of J (k_tabu_int), row pitch ldj
    int ldj;
    const int32_t *rp, *ci;
    const int32_t *amb;
    const int8_t *spins;
    const double *h_eff;
    int8_t *spins_out;    // read-out with the best configuration merged in
    double *d_best;
};

__device__ __forceinline__ double tabu_j(const TabuArgs &a, int i, int j) {
    if (!a.csr) return a.J[(int64_t)i * a.N + j];
    int lo = a.rp[i], hi = a.rp[i + 1];
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a.ci[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    return (lo < a.rp[i + 1] && a.ci[lo] == j) ? a.J[lo] : 0.0;
}

// Minimum over the wavefront, in every lane: quad xor 1 and 2, the half-row mirror (lane i
// with 7 - i) and the row mirror (i with 15 - i), then the permlane swaps across rows.
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    return __hiloint2double(dpp_i32<CTRL>(__double2hiint(x)), dpp_i32<CTRL>(__double2loint(x)));
}
__device__ __forceinline__ int wave_min_i32(int x) {
    x = min(x, dpp_i32<0xB1>(x));
    x = min(x, dpp_i32<0x4E>(x));
    x = min(x, dpp_i32<0x141>(x));
    x = min(x, dpp_i32<0x140>(x));
    const auto p = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    x = min((int)p[0], (int)p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    return min((int)q[0], (int)q[1]);
}
template <bool ROW32>
__device__ __forceinline__ double swap_min_f64(double x) {
    const unsigned lo = (unsigned)__double2loint(x), hi = (unsigned)__double2hiint(x);
    const auto l = ROW32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                         : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = ROW32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                         : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return fmin(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
}
// NaN gains are never the minimum (fmin returns the number).
__device__ __forceinline__ double wave_min_f64(double x) {
    x = fmin(x, dpp_f64<0xB1>(x));
    x = fmin(x, dpp_f64<0x4E>(x));
    x = fmin(x, dpp_f64<0x141>(x));
    x = fmin(x, dpp_f64<0x140>(x));
    x = swap_min_f64<false>(x);
    return swap_min_f64<true>(x);
}

// Minimum over NW (2 .. 16) slots that lane v holds as slot v mod NW.
template <int NW>
__device__ __forceinline__ int slots_min_i32(int x) {
    x = min(x, dpp_i32<0xB1>(x));
    if (NW > 2) x = min(x, dpp_i32<0x4E>(x));
    if (NW > 4) x = min(x, dpp_i32<0x141>(x));
    if (NW > 8) x = min(x, dpp_i32<0x140>(x));
    return x;
}
template <int NW>
__device__ __forceinline__ double slots_min_f64(double x) {
    x = fmin(x, dpp_f64<0xB1>(x));
    if (NW > 2) x = fmin(x, dpp_f64<0x4E>(x));
    if (NW > 4) x = fmin(x, dpp_f64<0x141>(x));
    if (NW > 8) x = fmin(x, dpp_f64<0x140>(x));
    return x;
}

enum { TABU_MAXN = 4096 };

// Spins a = tid + TPB k, k < SPT.
template <int TPB, int SPT>
__global__ __launch_bounds__(TPB) void k_tabu(TabuArgs a) {
    constexpr int NW = TPB / 64;
    __shared__ int8_t sx[TPB * SPT];            // starting spins of the ambivalent set
    __shared__ int32_t sA[TPB * SPT];           // their indices
    __shared__ double sd[2][NW];
    __shared__ int2 sk[2][NW];                  // (2 a + [x_a > 0], index of spin a)
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n = a.n, N = a.N;
    const int32_t *A = a.amb + (int64_t)r * n;
    const int8_t *s0 = a.spins + (int64_t)r * N;
    for (int b = tid; b < n; b += TPB) {
        const int i = A[b];
        sA[b] = i;
        sx[b] = s0[i];
    }
    __syncthreads();
    double f[SPT];
    int x[SPT], xb[SPT], Ai[SPT];
    int64_t until[SPT];
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        const int ai = tid + TPB * k;
        f[k] = 0.0; x[k] = 1; xb[k] = 1; Ai[k] = 0; until[k] = 0;
        if (ai < n) {
            Ai[k] = sA[ai];
            x[k] = xb[k] = sx[ai];
            f[k] = a.h_eff[(int64_t)r * n + ai];
        }
    }
    // the loads of a row are independent, so several are in flight; each sum keeps the
    // order b = 0, 1, ...
    if (!a.csr) {
#pragma unroll 8
        for (int b = 0; b < n; b++) {
            const int col = sA[b];
            const double xd = (double)sx[b];
#pragma unroll
            for (int k = 0; k < SPT; k++) {
                const double J = a.J[(int64_t)Ai[k] * N + col];
                if (b != tid + TPB * k) f[k] = f[k] + J * xd;
            }
        }
    } else {
        for (int b = 0; b < n; b++)
#pragma unroll
            for (int k = 0; k < SPT; k++)
                if (tid + TPB * k < n && b != tid + TPB * k)
                    f[k] = f[k] + tabu_j(a, Ai[k], sA[b]) * (double)sx[b];
    }
    const int tenure = min(a.tenure, n - 1);
    double D = 0.0, Db = 0.0;
    for (int64_t t = 1; t <= a.iters; t++) {
        const int par = (int)(t & 1);
        double bd = INFINITY;
        int2 bk = make_int2(INT_MAX, 0);
#pragma unroll
        for (int k = 0; k < SPT; k++) {        // ascending index: the first of equals stays
            const int ai = tid + TPB * k;
            const double d = x[k] > 0 ? -2.0 * f[k] : 2.0 * f[k];
            if (ai < n && (until[k] < t || D + d < Db) && (d < bd || (d == bd && bk.x == INT_MAX))) {
                bd = d;
                bk = make_int2(2 * ai + (x[k] > 0), Ai[k]);
            }
        }
        const double m = wave_min_f64(bd);
        // the owner of the wavefront's best: the smallest index among the lanes that hold it
        const bool tied = bd == m && bk.x != INT_MAX;
        const uint64_t mask = __ballot(tied);
        bool own = tied;
        if (mask & (mask - 1)) {   // uniform: the minimum needs every lane
            const int first = wave_min_i32(tied ? bk.x : INT_MAX);
            own = tied && bk.x == first;
        }
        if (NW == 1) {
            // all in registers: the owner's lane is broadcast
            const int src = mask ? __ffsll((unsigned long long)__ballot(own)) - 1 : 0;
            bk.x = __builtin_amdgcn_readlane(bk.x, src);
            bk.y = __builtin_amdgcn_readlane(bk.y, src);
            bd = m;
        } else {
            if (own || (mask == 0 && lane == 0)) { sd[par][w] = bd; sk[par][w] = bk; }
            __syncthreads();
            // lane v takes slot v mod NW
            bd = sd[par][lane & (NW - 1)];
            bk = sk[par][lane & (NW - 1)];
            const double mm = slots_min_f64<NW>(bd);
            const bool tied2 = bd == mm && bk.x != INT_MAX;
            uint64_t mask2 = __ballot(tied2) & ((1ull << NW) - 1ull);
            if (mask2 & (mask2 - 1)) {
                const int first = wave_min_i32(tied2 ? bk.x : INT_MAX);
                mask2 = __ballot(tied2 && bk.x == first);
            }
            const int src = mask2 ? __ffsll((unsigned long long)mask2) - 1 : 0;
            bk.x = __builtin_amdgcn_readlane(bk.x, src);
            bk.y = __builtin_amdgcn_readlane(bk.y, src);
            bd = mm;
        }
        const int bi = bk.x >> 1, bo = (bk.x & 1) ? 1 : -1;
        // At most tenure < n spins are tabu, so some move is allowed; only gains that
        // are all NaN (fields overflowed) leave none.  bi is the same in every thread.
        if (bk.x == INT_MAX) break;
        D = D + bd;
        const int rowj = __builtin_amdgcn_readfirstlane(bk.y);
        double J[SPT];
#pragma unroll
        for (int k = 0; k < SPT; k++) J[k] = tid + TPB * k < n ? tabu_j(a, rowj, Ai[k]) : 0.0;
#pragma unroll
        for (int k = 0; k < SPT; k++) {
            const int ai = tid + TPB * k;
            if (ai == bi) {
                x[k] = -x[k];
                until[k] = t + tenure;
            } else {
                f[k] = f[k] - (bo > 0 ? 2.0 * J[k] : -2.0 * J[k]);
            }
        }
        if (D < Db) {   // uniform
            Db = D;
#pragma unroll
            for (int k = 0; k < SPT; k++) xb[k] = x[k];
        }
    }
    int8_t *so_r = a.spins_out + (int64_t)r * N;
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        const int ai = tid + TPB * k;
        if (ai < n) so_r[Ai[k]] = (int8_t)xb[k];
    }
    if (tid == 0) a.d_best[r] = Db;
}

// Integral coupling (i, j) from the storage JT (JT_BIT here: the binary64 J).
template <int JT>
__device__ __forceinline__ int tabu_ji(const TabuArgs &a, const uint8_t *row, int j) {
    if constexpr (JT == JT_FP8) {
        const uint32_t b = row[j];
        return (int)__builtin_amdgcn_cvt_f32_fp8((int)b, 0);
    } else if constexpr (JT == JT_BF16) {
        return (int)__uint_as_float((uint32_t)((const uint16_t *)row)[j] << 16);
    } else if constexpr (JT == JT_F32) {
        return (int)((const float *)row)[j];
    } else {
        return (int)((const double *)row)[j];
    }
}

template <int JT>
__device__ __forceinline__ const uint8_t *tabu_row(const TabuArgs &a, int i) {
    constexpr int esz = JT == JT_FP8 ? 1 : JT == JT_BF16 ? 2 : JT == JT_F32 ? 4 : 8;
    return (const uint8_t *)(JT == JT_BIT ? (const void *)a.J : a.Js) +
           (int64_t)i * (JT == JT_BIT ? a.N : a.ldj) * esz;
}

// Dense integral instances with 2 (N + 1) max(|J|, |h|) below 2^16 (see launch_tabu).  d[k]
// holds the gain -2 x f; a flip of b adds 4 x_a x_b J_ab to the others and negates its own.
template <int TPB, int SPT, int JT>
__global__ __launch_bounds__(TPB) void k_tabu_int(TabuArgs a) {
    constexpr int NW = TPB / 64;
    __shared__ int8_t sx[TPB * SPT];
    __shared__ int32_t sA[TPB * SPT];
    __shared__ __align__(16) int2 sk[2][NW];    // (key, index of its spin)
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n = a.n, N = a.N;
    const int32_t *A = a.amb + (int64_t)r * n;
    const int8_t *s0 = a.spins + (int64_t)r * N;
    for (int b = tid; b < n; b += TPB) {
        const int i = A[b];
        sA[b] = i;
        sx[b] = s0[i];
    }
    __syncthreads();
    int d[SPT], x[SPT], xb[SPT], Ai[SPT], until[SPT];
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        const int ai = tid + TPB * k;
        d[k] = 0; x[k] = xb[k] = 1; Ai[k] = 0; until[k] = 0;
        if (ai < n) {
            Ai[k] = sA[ai];
            x[k] = xb[k] = sx[ai];
            d[k] = (int)a.h_eff[(int64_t)r * n + ai];
        }
    }
    // d holds f_a here: J is symmetric, so row b is read along the threads' columns
#pragma unroll 8
    for (int b = 0; b < n; b++) {
        const uint8_t *row = tabu_row<JT>(a, sA[b]);
        const int xs = sx[b];
#pragma unroll
        for (int k = 0; k < SPT; k++) {
            const int J = tabu_ji<JT>(a, row, Ai[k]);
            d[k] += b != tid + TPB * k ? J * xs : 0;
        }
    }
#pragma unroll
    for (int k = 0; k < SPT; k++) d[k] = -2 * x[k] * d[k];
    const int tenure = min(a.tenure, n - 1);
    int D = 0, Db = 0;
    for (int t = 1; t <= (int)a.iters; t++) {
        const int par = t & 1;
        int key = INT_MAX, ka = 0;
#pragma unroll
        for (int k = 0; k < SPT; k++) {
            const int ai = tid + TPB * k;
            const int kk = (d[k] << 13) + 2 * ai + (x[k] > 0);
            if (ai < n && (until[k] < t || D + d[k] < Db) && kk < key) {
                key = kk;
                ka = Ai[k];
            }
        }
        const int m = wave_min_i32(key);
        int2 bk;
        if (NW == 1) {
            const uint64_t mask = __ballot(key == m);      // keys are distinct
            bk.x = m;
            bk.y = __builtin_amdgcn_readlane(ka, __ffsll((unsigned long long)mask) - 1);
        } else {
            if (key == m) sk[par][w] = make_int2(key, ka);
            __syncthreads();
            bk = sk[par][lane & (NW - 1)];
            const int mm = slots_min_i32<NW>(bk.x);
            bk.y = __builtin_amdgcn_readlane(bk.y, __ffsll((unsigned long long)__ballot(bk.x == mm)) - 1);
            bk.x = mm;
        }
        const int key1 = __builtin_amdgcn_readfirstlane(bk.x);
        if (key1 == INT_MAX) break;                        // not reached: tenure < n
        const int bi = (key1 >> 1) & (TABU_MAXN - 1), bo4 = (key1 & 1) ? 4 : -4;
        D += key1 >> 13;
        const uint8_t *row = tabu_row<JT>(a, __builtin_amdgcn_readfirstlane(bk.y));
        int J[SPT];
#pragma unroll
        for (int k = 0; k < SPT; k++) J[k] = tabu_ji<JT>(a, row, Ai[k]);
#pragma unroll
        for (int k = 0; k < SPT; k++) {
            if (tid + TPB * k == bi) {
                x[k] = -x[k];
                d[k] = -d[k];
                until[k] = t + tenure;
            } else {
                d[k] += x[k] * (bo4 * J[k]);
            }
        }
        if (D < Db) {   // uniform
            Db = D;
#pragma unroll
            for (int k = 0; k < SPT; k++) xb[k] = x[k];
        }
    }
    int8_t *so_r = a.spins_out + (int64_t)r * N;
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        const int ai = tid + TPB * k;
        if (ai < n) so_r[Ai[k]] = (int8_t)xb[k];
    }
    if (tid == 0) a.d_best[r] = (double)Db;
}

template <int TPB, int SPT>
static void launch_tabu_int(const TabuArgs &a, int jt, hipStream_t st) {
    switch (jt) {
        case JT_FP8: k_tabu_int<TPB, SPT, JT_FP8><<<a.R, TPB, 0, st>>>(a); break;
        case JT_BF16: k_tabu_int<TPB, SPT, JT_BF16><<<a.R, TPB, 0, st>>>(a); break;
        case JT_F32: k_tabu_int<TPB, SPT, JT_F32><<<a.R, TPB, 0, st>>>(a); break;
        default: k_tabu_int<TPB, SPT, JT_BIT><<<a.R, TPB, 0, st>>>(a); break;
    }
}

hipError_t launch_tabu(const Instance &I, int R, int n, const int32_t *amb, const int8_t *spins,
                       const double *h_eff, int64_t iters, int tenure, int8_t *spins_out,
                       double *d_best, hipStream_t st) {
    TabuArgs a;
    a.N = I.N; a.R = R; a.n = n; a.csr = I.layout == HQA_CSR; a.tenure = tenure; a.iters = iters;
    a.J = I.J64; a.rp = I.rp; a.ci = I.ci; a.amb = amb; a.spins = spins; a.h_eff = h_eff;
    a.spins_out = spins_out; a.d_best = d_best;
    a.Js = nullptr; a.ldj = 0;
    if (R == 0 || n == 0) return hipSuccess;
    // |f_a| <= (N + 1) 2^(msb + 1): gains below 2^17 leave 13 bits of a signed word to the
    // index, |D| <= 2 (N + 1)^2 2^(msb + 1) stays below 2^31, and moves are counted in 32 bits
    const double big = I.es.lsb != INT32_MIN ? std::ldexp((double)I.N + 1.0, I.es.msb + 2) : 1e300;
    const bool ints = !a.csr && I.j_integral && big < 65536.0 &&
                      big * ((double)I.N + 1.0) < 2147483648.0 && iters < (1ll << 30);
    if (ints) {
        int jt = JT_BIT;
        if (I.js_exact && I.Js) {
            jt = (int)I.jt;
            a.Js = I.Js;
            a.ldj = I.Np;
        }
        if (n <= 64) launch_tabu_int<64, 1>(a, jt, st);
        else if (n <= 128) launch_tabu_int<128, 1>(a, jt, st);
        else if (n <= 256) launch_tabu_int<256, 1>(a, jt, st);
        else if (n <= 512) launch_tabu_int<512, 1>(a, jt, st);
        else if (n <= 1024) launch_tabu_int<512, 2>(a, jt, st);
        else if (n <= 2048) launch_tabu_int<512, 4>(a, jt, st);
        else launch_tabu_int<1024, 4>(a, jt, st);
    } else {
        if (n <= 64) k_tabu<64, 1><<<R, 64, 0, st>>>(a);
        else if (n <= 128) k_tabu<128, 1><<<R, 128, 0, st>>>(a);
        else if (n <= 256) k_tabu<256, 1><<<R, 256, 0, st>>>(a);
        else if (n <= 512) k_tabu<512, 1><<<R, 512, 0, st>>>(a);
        else if (n <= 1024) k_tabu<512, 2><<<R, 512, 0, st>>>(a);
        else if (n <= 2048) k_tabu<512, 4><<<R, 512, 0, st>>>(a);
        else k_tabu<1024, 4><<<R, 1024, 0, st>>>(a);
    }
    return hipGetLastError();
}

}  // namespace hqa
