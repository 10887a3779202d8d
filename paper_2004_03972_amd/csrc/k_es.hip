// k_es.hip -- learned early stop: per-spin features from the MD statistics, a
// 12-64-64-3 GELU perceptron (forward, class-weighted cross-entropy gradient,
// Adam), and the spin read-out driven by predicted labels.
//
// The paper defines no learned component; the definitions are the library's:
// statistics over a window of steps [K0, K1) (nine running sums per spin and
// replica, accumulated in the MD step epilogue), twelve features at the
// checkpoint normalised per replica, three classes {frozen +, frozen -,
// ambivalent}.  Parameter vector (5187 binary32): W1[64][12], b1[64],
// W2[64][64], b2[64], W3[3][64], b3[3], weights row-major [out][in].
#include <math.h>

#include <algorithm>

#include "hqa_internal.h"

namespace hqa {

enum { NF = 12, H1 = 64, H2 = 64, NC = 3 };
enum { OFF_W1 = 0, OFF_B1 = OFF_W1 + H1 * NF, OFF_W2 = OFF_B1 + H1, OFF_B2 = OFF_W2 + H2 * H1,
       OFF_W3 = OFF_B2 + H2, OFF_B3 = OFF_W3 + NC * H2, NPARAM = OFF_B3 + NC };

// ---------------------------------------------------------------- row norms
__global__ void k_row_norms(const double *J, const int32_t *rp, const int32_t *ci, int N, int csr,
                            float *n1, float *inv_n2) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    double a = 0.0, b = 0.0;
    if (!csr) {
        for (int j = 0; j < N; j++) {
            double v = J[(int64_t)i * N + j];
            a += fabs(v);
            b += v * v;
        }
    } else {
        for (int e = rp[i]; e < rp[i + 1]; e++) {
            a += fabs(J[e]);
            b += J[e] * J[e];
        }
    }
    n1[i] = (float)a;
    inv_n2[i] = b > 0.0 ? (float)(1.0 / sqrt(b)) : 0.0f;
}

hipError_t launch_row_norms(const Instance &I, float *n1, float *inv_n2, hipStream_t st) {
    k_row_norms<<<(I.N + 255) / 256, 256, 0, st>>>(I.J64, I.rp, I.ci, I.N, I.layout == HQA_CSR,
                                                   n1, inv_n2);
    return hipGetLastError();
}

// ------------------------------------------------------------------ features
struct FeatArgs {
    int N, R, ld, smaj;
    int64_t sst;
    float K, tau, mean_n1;
    const float *phi, *st, *n1;
    float *scale;         // [R][2], behind the statistics
    float *feat;
};

__device__ __forceinline__ int64_t fidx(const FeatArgs &a, int r, int i) {
    return a.smaj ? (int64_t)i * a.ld + r : (int64_t)r * a.ld + i;
}

// The features of one spin and replica (position k of the state).
__device__ __forceinline__ void feature_row(const FeatArgs &a, int64_t k, int i, float sig, float pmean,
                                            float *f) {
    const float *S = a.st + k;
    const float m0 = S[0] / a.K, m5 = S[5 * a.sst] / a.K;
    f[0] = m0 / sig;
    f[1] = sqrtf(fmaxf(S[1 * a.sst] / a.K - m0 * m0, 0.f)) / sig;
    f[2] = (S[2 * a.sst] / a.K) / sig;
    f[3] = a.phi[k] / sig;
    f[4] = fabsf(2.f * S[3 * a.sst] / a.K - 1.f);
    f[5] = S[4 * a.sst] / a.K;
    f[6] = m5 / sig;
    f[7] = sqrtf(fmaxf(S[6 * a.sst] / a.K - m5 * m5, 0.f)) / sig;
    f[8] = (S[7 * a.sst] / a.K) / sig;
    f[9] = (S[8 * a.sst] / a.K) / pmean;
    f[10] = a.mean_n1 > 0.f ? a.n1[i] / a.mean_n1 : 0.f;
    f[11] = a.tau;
}

__global__ __launch_bounds__(256) void k_features(FeatArgs a) {
    __shared__ float red[2][256];
    const int r = blockIdx.x, tid = threadIdx.x;
    float s2 = 0.f, pm = 0.f;
    for (int i = tid; i < a.N; i += 256) {
        const int64_t k = fidx(a, r, i);
        const float x = a.phi[k];
        s2 += x * x;
        pm += a.st[8 * a.sst + k] / a.K;
    }
    red[0][tid] = s2;
    red[1][tid] = pm;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
            red[0][tid] += red[0][tid + s];
            red[1][tid] += red[1][tid + s];
        }
        __syncthreads();
    }
    float sig = sqrtf(red[0][0] / (float)a.N);
    if (sig == 0.f) sig = 1.f;
    float pmean = red[1][0] / (float)a.N;
    if (pmean == 0.f) pmean = 1.f;
    for (int i = tid; i < a.N; i += 256) {
        const int64_t k = fidx(a, r, i);
        feature_row(a, k, i, sig, pmean, a.feat + ((int64_t)r * a.N + i) * NF);
    }
}

// Replica-minor state: four replicas a workgroup, lane group t / 4 = 0 .. 255 taking the spins of
// thread t / 4 of k_features, so that every sum has the same terms in the same order; the two
// scales go to a.scale[2 r], [2 r + 1].
__global__ __launch_bounds__(1024) void k_feature_scales(FeatArgs a) {
    __shared__ float red[2][256][5];
    const int q = threadIdx.x & 3, j = threadIdx.x >> 2, r = blockIdx.x * 4 + q;
    float s2 = 0.f, pm = 0.f;
    if (r < a.R)
#pragma unroll 4
        for (int i = j; i < a.N; i += 256) {
            const int64_t k = (int64_t)i * a.ld + r;
            const float x = a.phi[k];
            s2 += x * x;
            pm += a.st[8 * a.sst + k] / a.K;
        }
    red[0][j][q] = s2;
    red[1][j][q] = pm;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (j < s) {
            red[0][j][q] += red[0][j + s][q];
            red[1][j][q] += red[1][j + s][q];
        }
        __syncthreads();
    }
    if (j == 0 && r < a.R) {
        float sig = sqrtf(red[0][0][q] / (float)a.N), pmean = red[1][0][q] / (float)a.N;
        a.scale[2 * r] = sig == 0.f ? 1.f : sig;
        a.scale[2 * r + 1] = pmean == 0.f ? 1.f : pmean;
    }
}

// ... and the features of 16 spins x 32 replicas a workgroup, read along the replicas and turned
// in LDS to rows of 16 spins.  Bound by the ten arrays read and the twelve written; N = 10^4,
// R = 128: 236 us as one workgroup a replica reading across the lines, 53 both kernels.
__global__ __launch_bounds__(512) void k_features_turn(FeatArgs a) {
    __shared__ float t[32][16 * NF + 1];
    const int tid = threadIdx.x, x = tid & 31, y = tid >> 5;
    const int i0 = blockIdx.x * 16, r0 = blockIdx.y * 32, i = i0 + y, r = r0 + x;
    if (i < a.N && r < a.R) {
        const int64_t k = (int64_t)i * a.ld + r;
        feature_row(a, k, i, a.scale[2 * r], a.scale[2 * r + 1], &t[x][y * NF]);
    }
    __syncthreads();
    const int cols = min(16, a.N - i0) * NF;
    for (int e = tid; e < 32 * 16 * NF; e += 512) {
        const int rr = e / (16 * NF), c = e % (16 * NF);
        if (c < cols && r0 + rr < a.R) a.feat[((int64_t)(r0 + rr) * a.N + i0) * NF + c] = t[rr][c];
    }
}

hipError_t launch_features(const Instance &I, int R, int64_t K, float tau, float mean_n1,
                           float *feat, hipStream_t st) {
    FeatArgs a;
    a.N = I.N; a.R = R; a.ld = I.ld; a.smaj = I.smaj;
    a.sst = I.smaj ? (int64_t)I.N * I.ld : (int64_t)I.Rp * I.ld;
    a.K = (float)K; a.tau = tau; a.mean_n1 = mean_n1;
    a.phi = I.phi32[I.cur]; a.st = I.st; a.n1 = I.n1; a.feat = feat;
    a.scale = I.st + 9 * a.sst;
    if (I.smaj && features_turn_fits(I.N, R)) {
        k_feature_scales<<<(R + 3) / 4, 1024, 0, st>>>(a);
        k_features_turn<<<dim3((I.N + 15) / 16, (R + 31) / 32), 512, 0, st>>>(a);
        return hipGetLastError();
    }
    k_features<<<R, 256, 0, st>>>(a);
    return hipGetLastError();
}

// -------------------------------------------------------------------- MLP
__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float rbf(float x, bool on) { return on ? (float)(bf16)x : x; }

__device__ __forceinline__ uint64_t mix64(uint64_t seed, uint64_t ctr) {
    uint64_t z = seed + (ctr + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Weights uniform in [-1/sqrt(fan_in), 1/sqrt(fan_in)] from the counter hash, biases 0.
__global__ void k_mlp_init(float *P, uint64_t seed) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= NPARAM) return;
    int fan = 0;
    if (k < OFF_B1) fan = NF;
    else if (k >= OFF_W2 && k < OFF_B2) fan = H1;
    else if (k >= OFF_W3 && k < OFF_B3) fan = H2;
    if (!fan) { P[k] = 0.f; return; }
    double u = (double)(mix64(seed, (uint64_t)k) >> 11) * (1.0 / 9007199254740992.0);
    P[k] = (float)((2.0 * u - 1.0) / sqrt((double)fan));
}

hipError_t launch_mlp_init(float *P, uint64_t seed, hipStream_t st) {
    k_mlp_init<<<(NPARAM + 255) / 256, 256, 0, st>>>(P, seed);
    return hipGetLastError();
}

// The perceptron runs on 16x16x4 binary32 MFMAs, 16 samples a tile.  A layer is
// D = W X: the A operand holds 16 outputs (row = lane mod 16) x 4 inputs (column = lane
// group g = lane / 16), the B operand 4 inputs x 16 samples (sample = lane mod 16), and
// accumulator v of a lane is output 4 g + v of its sample.  This MFMA adds its four
// products one after another in ascending input order, each by a fused multiply-add, and
// the accumulator starts at the bias, so a layer's sums are those of a scalar fmaf loop
// over the inputs, bit for bit.  Activations come out as outputs 4 g + v and go in as
// inputs 4 c + g: a 4 x 4 transpose between the lane groups and four registers.
enum { MLP_TILE = 16, LP = 68 };   // LP: pitch of a 64-unit row in LDS, every bank once per operand

// v[j] of lane group g: element 4 g + j in, element 4 j + g out.
__device__ __forceinline__ void group_transpose(f32x4 &v) {
    unsigned a[4];
#pragma unroll
    for (int j = 0; j < 4; j++) a[j] = __float_as_uint(v[j]);
    const auto p02 = __builtin_amdgcn_permlane32_swap(a[0], a[2], false, false);
    const auto p13 = __builtin_amdgcn_permlane32_swap(a[1], a[3], false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(p02[0], p13[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(p02[1], p13[1], false, false);
    v[0] = __uint_as_float(lo[0]);
    v[1] = __uint_as_float(lo[1]);
    v[2] = __uint_as_float(hi[0]);
    v[3] = __uint_as_float(hi[1]);
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void softmax3(const float (&z3)[NC], float (&pr)[NC]) {
    float mx = -INFINITY, den = 0.f, e[NC];
#pragma unroll
    for (int o = 0; o < NC; o++) mx = fmaxf(mx, z3[o]);
#pragma unroll
    for (int o = 0; o < NC; o++) { e[o] = expf(z3[o] - mx); den += e[o]; }
#pragma unroll
    for (int o = 0; o < NC; o++) pr[o] = e[o] / den;
}

// Inference.  The weights of layers 2 and 3 sit in LDS, a wavefront takes S tiles at a time
// (S = 4: the softmax then has a sample in every lane; S = 1 spreads few samples over more
// wavefronts).  BF: BF16 inference (weights and layer inputs rounded to bfloat16, binary32
// accumulation).  Bound by the vector units: 128 erff per sample, about 1400 vector
// instructions per tile of 16 against 92 MFMAs, so four wavefronts per SIMD overlap the two.
// Measured, 1.28e6 samples in BF16: a thread per sample (weights read through the caches for
// every sample) 950 us; all weights in registers, two wavefronts per SIMD, 250 us; this
// kernel 220 us.  8192 samples: 7.4 us.
template <bool BF, int S>
__global__ __launch_bounds__(256, 4) void k_mlp_predict(const float *P, int64_t B, const float *x,
                                                        float *prob) {
    __shared__ __align__(16) float sm2[H2 * LP], sm3[16 * LP], smb[H1 + H2 + 16];
    const int tid = threadIdx.x, lane = tid & 63, kg = lane >> 4, l16 = lane & 15;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const float4 q = *(const float4 *)(P + OFF_W2 + 4 * (tid + 256 * j));
        *(float4 *)&sm2[((tid + 256 * j) >> 4) * LP + 4 * (tid & 15)] =
            make_float4(rbf(q.x, BF), rbf(q.y, BF), rbf(q.z, BF), rbf(q.w, BF));
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int o = (tid + 256 * j) >> 6, i = tid & 63;
        sm3[o * LP + i] = o < NC ? rbf(P[OFF_W3 + o * H2 + i], BF) : 0.f;
    }
    if (tid < H1 + H2 + 16)
        smb[tid] = tid < H1 ? P[OFF_B1 + tid] : tid < H1 + H2 ? P[OFF_B2 + tid - H1]
                   : tid < H1 + H2 + NC ? P[OFF_B3 + tid - H1 - H2] : 0.f;
    float w1[4][NF / 4];
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
        for (int c = 0; c < NF / 4; c++) w1[t][c] = rbf(P[OFF_W1 + (16 * t + l16) * NF + 4 * c + kg], BF);
    __syncthreads();
    const int64_t groups = (B + MLP_TILE * S - 1) / (MLP_TILE * S);
    for (int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); g < groups; g += (int64_t)gridDim.x * 4) {
        f32x4 z3[S];
#pragma unroll 1
        for (int s = 0; s < S; s++) {
            const float *xs = x + min(g * MLP_TILE * S + 16 * s + l16, B - 1) * NF;
            f32x4 h[4], u[4];
            // the weights are read from LDS tile by tile: an offset the compiler cannot see
            // through keeps it from holding all of them in (too many) registers
            int at = 0;
            asm volatile("" : "+v"(at));
            const float *p2 = sm2 + l16 * LP + kg + at, *p3 = sm3 + l16 * LP + kg + at;
            const float *pb = smb + 4 * kg + at;
#pragma unroll
            for (int t = 0; t < 4; t++) h[t] = *(const f32x4 *)&pb[16 * t];
#pragma unroll
            for (int c = 0; c < NF / 4; c++) {
                const float xi = rbf(xs[4 * c + kg], BF);
#pragma unroll
                for (int t = 0; t < 4; t++) h[t] = mfma4(w1[t][c], xi, h[t]);
            }
#pragma unroll
            for (int t = 0; t < 4; t++) {
#pragma unroll
                for (int v = 0; v < 4; v++) h[t][v] = rbf(gelu(h[t][v]), BF);
                group_transpose(h[t]);
                u[t] = *(const f32x4 *)&pb[H1 + 16 * t];
            }
#pragma unroll
            for (int c = 0; c < H1 / 4; c++)
#pragma unroll
                for (int t = 0; t < 4; t++)
                    u[t] = mfma4(p2[16 * t * LP + 4 * c], h[c >> 2][c & 3], u[t]);
            f32x4 z = *(const f32x4 *)&pb[H1 + H2];
#pragma unroll
            for (int t = 0; t < 4; t++) {
#pragma unroll
                for (int v = 0; v < 4; v++) u[t][v] = rbf(gelu(u[t][v]), BF);
                group_transpose(u[t]);
#pragma unroll
                for (int j = 0; j < 4; j++) z = mfma4(p3[16 * t + 4 * j], u[t][j], z);
            }
            // the S tiles' outputs sit in lane group 0; group s takes tile s
#pragma unroll
            for (int k = 0; k < S; k++)
                if (k == s) z3[k] = z;
        }
        float zz[NC], pr[NC];
        if constexpr (S == 4) {
#pragma unroll
            for (int o = 0; o < NC; o++) {
                const auto p02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z3[0][o]), __float_as_uint(z3[2][o]), false, false);
                const auto p13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z3[1][o]), __float_as_uint(z3[3][o]), false, false);
                zz[o] = __uint_as_float(__builtin_amdgcn_permlane16_swap(p02[0], p13[0], false, false)[0]);
            }
        } else {
#pragma unroll
            for (int o = 0; o < NC; o++) zz[o] = z3[0][o];
        }
        softmax3(zz, pr);
        const int64_t out = g * MLP_TILE * S + lane;
        if (lane < MLP_TILE * S && out < B) {
#pragma unroll
            for (int o = 0; o < NC; o++) prob[out * NC + o] = pr[o];
        }
    }
}

template <int S>
static void launch_predict(const float *P, int64_t B, const float *x, float *prob, int bf, hipStream_t st) {
    const int64_t groups = (B + MLP_TILE * S - 1) / (MLP_TILE * S);
    const unsigned grid = (unsigned)std::min<int64_t>((groups + 3) / 4, 1024);   // four workgroups per CU
    if (bf) k_mlp_predict<true, S><<<grid, 256, 0, st>>>(P, B, x, prob);
    else k_mlp_predict<false, S><<<grid, 256, 0, st>>>(P, B, x, prob);
}

hipError_t launch_mlp_predict(const float *P, int64_t B, const float *x, float *prob, int bf,
                              hipStream_t st) {
    if (B == 0) return hipSuccess;
    // below a tile for each of the 4096 resident wavefronts, one tile at a time is the
    // wider split
    if (B <= 4096 * MLP_TILE) launch_predict<1>(P, B, x, prob, bf, st);
    else launch_predict<4>(P, B, x, prob, bf, st);
    return hipGetLastError();
}

// Gradient of sum_s w_{y_s} * (-log prob_s[y_s]) (unnormalised), with the sum of the
// weighted losses and of the weights: each workgroup writes one partial of GP floats (its
// accumulators), added up in order by k_grad_reduce.
//
// A wavefront runs 16 samples forward and backward on MFMAs with the weights in LDS (W2
// both ways round, rows padded to 68 floats so that an operand read touches every bank
// once).  The parameter gradients contract over the samples, so their operands have the
// samples across the lane groups and the units across the lanes: activations and deltas
// pass through a per-wavefront LDS block [sample][unit] whose unit index is exclusive-ored
// with 16 (sample mod 4), free of conflicts both ways, and the products stay in
// accumulators for all tiles of the wavefront.  64 of the 256 MFMAs of a tile are W2's
// gradient.  Measured, 8192 samples: a thread per sample with one wavefront per CU 146 us
// and 14 us of clears, normalisation and Adam; this kernel 16 us and k_grad_reduce 4 us
// (524,288 samples: 243 and 9 us, 65 TFLOP/s).
enum { GF = 26, GP = GF * 256 };   // GF accumulators of 64 lanes x 4 in a partial
enum { L_W2 = 0, L_W2T = L_W2 + H2 * LP, L_W1 = L_W2T + H1 * LP, L_W3 = L_W1 + H1 * NF,
       L_W3T = L_W3 + 16 * LP, L_B1 = L_W3T + 4 * 80, L_B2 = L_B1 + H1, L_B3 = L_B2 + H2,
       L_END = L_B3 + 16 };
enum { W_BUF = 16 * 64, W_END = 2 * W_BUF + 64 };   // per wavefront: two blocks and the output deltas
static_assert(L_END + 4 * W_END >= 2 * GP, "the workgroup's gradient sum reuses all the LDS");

__device__ __forceinline__ int blk(int sample, int unit) { return sample * 64 + (unit ^ (16 * (sample & 3))); }

// Orders this wavefront's LDS writes before the reads of other lanes' values.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(256, 2) void k_mlp_grad(const float *P, int64_t B, const float *x,
                                                     const int32_t *y, const float *cw, float *part) {
    extern __shared__ float sm[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kg = lane >> 4, l16 = lane & 15;
    {
        // all loads first: one round trip for the weights
        float4 q2[4], q1, q3;
        float qb = 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++) q2[j] = *(const float4 *)(P + OFF_W2 + 4 * (tid + 256 * j));
        if (tid < H1 * NF / 4) q1 = *(const float4 *)(P + OFF_W1 + 4 * tid);
        q3 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (tid < NC * H2 / 4) q3 = *(const float4 *)(P + OFF_W3 + 4 * tid);
        if (tid < H1) qb = P[OFF_B1 + tid];
        else if (tid < H1 + H2) qb = P[OFF_B2 + tid - H1];
        else if (tid < H1 + H2 + NC) qb = P[OFF_B3 + tid - H1 - H2];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int o = (tid + 256 * j) >> 4, i = 4 * (tid & 15);
            *(float4 *)&sm[L_W2 + o * LP + i] = q2[j];
            sm[L_W2T + (i + 0) * LP + o] = q2[j].x;
            sm[L_W2T + (i + 1) * LP + o] = q2[j].y;
            sm[L_W2T + (i + 2) * LP + o] = q2[j].z;
            sm[L_W2T + (i + 3) * LP + o] = q2[j].w;
        }
        if (tid < H1 * NF / 4) *(float4 *)&sm[L_W1 + 4 * tid] = q1;
        const int o = tid >> 4, i = 4 * (tid & 15);        // rows NC .. 15 are zero
        *(float4 *)&sm[L_W3 + o * LP + i] = q3;
        if (o < 4) *(float4 *)&sm[L_W3T + o * 80 + i] = q3;
        if (tid < H1 + H2 + 16) sm[L_B1 + tid] = qb;       // b1, b2, b3 and zeros
    }
    __syncthreads();
    float *b0 = sm + L_END + w * W_END, *bq = b0 + W_BUF, *d3b = bq + W_BUF;

    f32x4 g1[4], g2[4][4], g3[4];
    float gb2[4] = {0.f, 0.f, 0.f, 0.f}, gb3 = 0.f, lsum = 0.f, wsum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; t++) {
        g1[t] = g3[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 4; u++) g2[t][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const int64_t tiles = (B + MLP_TILE - 1) / MLP_TILE;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + w; tile < tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t s0 = tile * MLP_TILE, s = s0 + l16;
        const bool live = s < B;
        f32x4 h[4], dg1[4], dg2[4];
        // forward; h = gelu(z) and its derivative share one erff
        auto act = [&](f32x4 &z, f32x4 &d) {
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const float zz = z[v], e = erff(zz * 0.70710678118654752f);
                z[v] = 0.5f * zz * (1.0f + e);
                d[v] = 0.5f * (1.0f + e) + zz * expf(-0.5f * zz * zz) * 0.39894228040143268f;
            }
        };
#pragma unroll
        for (int t = 0; t < 4; t++) h[t] = *(const f32x4 *)&sm[L_B1 + 16 * t + 4 * kg];
#pragma unroll
        for (int c = 0; c < NF / 4; c++) {
            const float xi = live ? x[s * NF + 4 * c + kg] : 0.f;
#pragma unroll
            for (int t = 0; t < 4; t++) h[t] = mfma4(sm[L_W1 + (16 * t + l16) * NF + 4 * c + kg], xi, h[t]);
        }
        f32x4 u[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            act(h[t], dg1[t]);
            *(f32x4 *)&b0[blk(l16, 16 * t + 4 * kg)] = h[t];
            group_transpose(h[t]);
            u[t] = *(const f32x4 *)&sm[L_B2 + 16 * t + 4 * kg];
        }
#pragma unroll
        for (int c = 0; c < H1 / 4; c++)
#pragma unroll
            for (int t = 0; t < 4; t++)
                u[t] = mfma4(sm[L_W2 + (16 * t + l16) * LP + 4 * c + kg], h[c >> 2][c & 3], u[t]);
        f32x4 z = *(const f32x4 *)&sm[L_B3 + 4 * kg];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            act(u[t], dg2[t]);
            *(f32x4 *)&bq[blk(l16, 16 * t + 4 * kg)] = u[t];
            group_transpose(u[t]);
#pragma unroll
            for (int j = 0; j < 4; j++)
                z = mfma4(sm[L_W3 + l16 * LP + 16 * t + 4 * j + kg], u[t][j], z);
        }
        // outputs 0 .. 2 of sample l16 in lane group 0
        const float z3[NC] = {z[0], z[1], z[2]};
        float pr[NC];
        softmax3(z3, pr);
        const int yy = live ? y[s] : 0;
        const float wt = live ? cw[yy] : 0.f;
        if (kg == 0) {
            if (live) { lsum += -wt * logf(yy == 0 ? pr[0] : yy == 1 ? pr[1] : pr[2]); wsum += wt; }
            f32x4 d3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int o = 0; o < NC; o++) d3[o] = wt * (pr[o] - (o == yy ? 1.f : 0.f));
            *(f32x4 *)&d3b[4 * l16] = d3;
        }
        wave_lds_sync();
        // W3's gradient, then the deltas of layer 2
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const float a = l16 < 4 ? d3b[4 * (4 * c + kg) + l16] : 0.f;   // entry 3 is zero
            gb3 += a;
#pragma unroll
            for (int t = 0; t < 4; t++) g3[t] = mfma4(a, bq[blk(4 * c + kg, 16 * t + l16)], g3[t]);
        }
        const float d3k = d3b[4 * l16 + kg];
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < 4; t++) {
            u[t] = mfma4(sm[L_W3T + kg * 80 + 16 * t + l16], d3k, (f32x4){0.f, 0.f, 0.f, 0.f});
#pragma unroll
            for (int v = 0; v < 4; v++) u[t][v] = u[t][v] * dg2[t][v];
            *(f32x4 *)&bq[blk(l16, 16 * t + 4 * kg)] = u[t];
        }
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 4; c++) {
            float a[4], hb[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                a[t] = bq[blk(4 * c + kg, 16 * t + l16)];
                hb[t] = b0[blk(4 * c + kg, 16 * t + l16)];
                gb2[t] += a[t];
            }
#pragma unroll
            for (int to = 0; to < 4; to++)
#pragma unroll
                for (int ti = 0; ti < 4; ti++) g2[to][ti] = mfma4(a[to], hb[ti], g2[to][ti]);
        }
        wave_lds_sync();
        // deltas of layer 1, then W1's gradient (input column 12 is 1: the biases' gradient)
#pragma unroll
        for (int t = 0; t < 4; t++) {
            group_transpose(u[t]);
            h[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int c = 0; c < H2 / 4; c++)
#pragma unroll
            for (int t = 0; t < 4; t++)
                h[t] = mfma4(sm[L_W2T + (16 * t + l16) * LP + 4 * c + kg], u[c >> 2][c & 3], h[t]);
#pragma unroll
        for (int t = 0; t < 4; t++) {
#pragma unroll
            for (int v = 0; v < 4; v++) h[t][v] = h[t][v] * dg1[t][v];
            *(f32x4 *)&b0[blk(l16, 16 * t + 4 * kg)] = h[t];
        }
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int64_t sc = s0 + 4 * c + kg;
            const float xb = l16 < NF ? (sc < B ? x[sc * NF + l16] : 0.f) : l16 == NF ? 1.f : 0.f;
#pragma unroll
            for (int t = 0; t < 4; t++) g1[t] = mfma4(b0[blk(4 * c + kg, 16 * t + l16)], xb, g1[t]);
        }
        wave_lds_sync();
    }
    // bias gradients and the scalars over the wavefront
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
#pragma unroll
        for (int t = 0; t < 4; t++) gb2[t] += __shfl_xor(gb2[t], o);
        gb3 += __shfl_xor(gb3, o);
    }
    for (int o = 8; o > 0; o >>= 1) {
        lsum += __shfl_xor(lsum, o);
        wsum += __shfl_xor(wsum, o);
    }
    // the wavefronts' sums meet in LDS as whole accumulators: 2 and 3 into 0 and 1, then 1
    // into 0, which writes the workgroup's partial in accumulator order
    f32x4 *F = (f32x4 *)sm;
    auto each = [&](auto f) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
#pragma unroll
            for (int u = 0; u < 4; u++) f(4 * t + u, g2[t][u]);
            f(16 + t, g1[t]);
            f(20 + t, g3[t]);
        }
        f32x4 e = {gb2[0], gb2[1], gb2[2], gb2[3]};
        f(24, e);
#pragma unroll
        for (int t = 0; t < 4; t++) gb2[t] = e[t];
        e = (f32x4){gb3, lsum, wsum, 0.f};
        f(25, e);
        gb3 = e[0]; lsum = e[1]; wsum = e[2];
    };
    __syncthreads();
    if (w >= 2) each([&](int k, f32x4 &g) { F[((w - 2) * GF + k) * 64 + lane] = g; });
    __syncthreads();
    if (w < 2) each([&](int k, f32x4 &g) { g += F[(w * GF + k) * 64 + lane]; });
    if (w == 1) each([&](int k, f32x4 &g) { F[(GF + k) * 64 + lane] = g; });
    __syncthreads();
    if (w == 0) {
        f32x4 *out = (f32x4 *)(part + (int64_t)blockIdx.x * GP);
        each([&](int k, f32x4 &g) { out[k * 64 + lane] = g + F[(GF + k) * 64 + lane]; });
    }
}

// Totals of the workgroups' partial gradients (fixed order), divided by the weight sum;
// acc[2] is the mean weighted loss.  With lr > 0 the Adam step (Kingma & Ba 2015) follows:
// m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2, P -= lr (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
// A workgroup takes 64 entries of the partials, its wavefronts a quarter of them each.
__global__ __launch_bounds__(256) void k_grad_reduce(const float *part, int nb, float *grad, float *acc,
                                                     float *P, float *m, float *v, int64_t t, float lr,
                                                     float b1, float b2, float eps) {
    __shared__ float sg[4][64], sw[4], sl[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int e = blockIdx.x * 64 + lane;
    // entry e: component j of accumulator a in lane ln, whose group and unit are g and l
    const int a = e >> 8, ln = (e >> 2) & 63, j = e & 3, g = ln >> 4, l = ln & 15;
    int k = -1;
    if (a < 16) k = OFF_W2 + (16 * (a >> 2) + 4 * g + j) * H1 + 16 * (a & 3) + l;
    else if (a < 20 && l < NF) k = OFF_W1 + (16 * (a - 16) + 4 * g + j) * NF + l;
    else if (a < 20 && l == NF) k = OFF_B1 + 16 * (a - 16) + 4 * g + j;
    else if (a >= 20 && a < 24 && g == 0 && j < NC) k = OFF_W3 + j * H2 + 16 * (a - 20) + l;
    else if (a == 24 && g == 0) k = OFF_B2 + 16 * j + l;
    else if (a == 25 && g == 0 && j == 0 && l < NC) k = OFF_B3 + l;
    float s = 0.f, ls = 0.f, ws = 0.f;
    if (k >= 0) {
#pragma unroll 8
        for (int b = w; b < nb; b += 4) s += part[(int64_t)b * GP + e];
    }
    for (int b = tid; b < nb; b += 256) {               // loss and weight sum: lane 0 of the last one
        ls += part[(int64_t)b * GP + 25 * 256 + 1];
        ws += part[(int64_t)b * GP + 25 * 256 + 2];
    }
    for (int o = 32; o > 0; o >>= 1) {
        ls += __shfl_xor(ls, o);
        ws += __shfl_xor(ws, o);
    }
    sg[w][lane] = s;
    if (lane == 0) { sl[w] = ls; sw[w] = ws; }
    __syncthreads();
    if (w) return;
    const float W = (sw[0] + sw[1]) + (sw[2] + sw[3]), L = (sl[0] + sl[1]) + (sl[2] + sl[3]);
    if (e == 0) acc[2] = W > 0.f ? L / W : 0.f;
    if (k < 0) return;
    s = (sg[0][lane] + sg[1][lane]) + (sg[2][lane] + sg[3][lane]);
    s = W > 0.f ? s / W : 0.f;
    grad[k] = s;
    if (lr > 0.f) {
        const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
        m[k] = b1 * m[k] + (1.f - b1) * s;
        v[k] = b2 * v[k] + (1.f - b2) * s * s;
        P[k] -= lr * (m[k] / c1) / (sqrtf(v[k] / c2) + eps);
    }
}

constexpr int GRAD_BLOCKS = 512;   // two workgroups per CU

static int grad_blocks(int64_t B) {
    const int64_t tiles = (B + MLP_TILE - 1) / MLP_TILE;
    return (int)std::min<int64_t>((tiles + 3) / 4, GRAD_BLOCKS);
}

// Bytes of `part`, enough for any batch (13.6 MB).
size_t mlp_grad_scratch_bytes() { return (size_t)GRAD_BLOCKS * GP * sizeof(float); }

// Gradient and loss of B >= 1 samples into grad and acc[2]; with lr > 0, Adam step t.
hipError_t launch_mlp_grad(float *P, int64_t B, const float *x, const int32_t *y, const float *cw,
                           float *grad, float *acc, float *part, float *m, float *v, int64_t t,
                           float lr, hipStream_t st) {
    const int nb = grad_blocks(B);
    k_mlp_grad<<<nb, 256, sizeof(float) * (L_END + 4 * W_END), st>>>(P, B, x, y, cw, part);
    k_grad_reduce<<<GP / 64, 256, 0, st>>>(part, nb, grad, acc, P, m, v, t, lr, 0.9f, 0.999f,
                                                      1e-8f);
    return hipGetLastError();
}

// ------------------------------------------------- read-out from predictions
// spins: +1 if P(frozen +) >= P(frozen -) else -1; selection key 1 - P(ambivalent)
// as non-negative binary32 (smallest key = most ambivalent).
__global__ void k_probs_to_keys(int64_t n, const float *prob, int8_t *spins, float *key) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const float *p = prob + t * NC;
    spins[t] = p[0] >= p[1] ? 1 : -1;
    key[t] = 1.0f - p[2];
}

hipError_t launch_probs_to_keys(int64_t n, const float *prob, int8_t *spins, float *key,
                                hipStream_t st) {
    k_probs_to_keys<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, prob, spins, key);
    return hipGetLastError();
}

}  // namespace hqa
