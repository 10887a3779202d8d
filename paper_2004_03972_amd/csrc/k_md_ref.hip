// k_md_ref.hip -- binary64 reference MD step, field and MD Hamiltonian.
//
// The step uses a fixed operation order (built with -ffp-contract=off):
//   u   = fma chain over the stored couplings of row i in ascending column order
//   v   = phi^(M-1) by M-2 successive multiplications
//   g   = u + (2 h) |phi|
//   F   = (alpha (M v)) + (beta g),  F = r_g F when r_g != 1
//   p   = p - F/2 at q = 0 (initial half step), p - F afterwards
//   phi = phi + (alpha_(2q+1) p)      (alpha_(2q+1) scaled by r_g when r_g != 1)
// following the leapfrog of Methods ("Leapfrog algorithm") on Eq. 3.
#include "hqa_internal.h"

namespace hqa {

struct RefArgs {
    int N, R, M, csr;
    int64_t T;
    int W;
    double r_g;
    const double *J;
    const int32_t *rp, *ci;
    const double *h;
    const double *a64, *b64;
    const double *phi_in;
    double *phi_out, *p, *S;
    int32_t *err;
};

__device__ __forceinline__ double ref_field(const RefArgs &a, int i, const double *x) {
    double u = 0.0;
    if (!a.csr) {
        const double *Ji = a.J + (int64_t)i * a.N;
        for (int j = 0; j < a.N; j++) u = fma(Ji[j], x[j], u);
    } else {
        for (int e = a.rp[i]; e < a.rp[i + 1]; e++) u = fma(a.J[e], x[a.ci[e]], u);
    }
    return u;
}

__device__ __forceinline__ double ref_force(const RefArgs &a, int i, const double *x, double al,
                                            double be) {
    double xi = x[i];
    double u = ref_field(a, i, x);
    double v = xi;
    for (int k = 0; k < a.M - 2; k++) v = v * xi;
    double g = u + (2.0 * a.h[i]) * fabs(xi);
    double F = (al * ((double)a.M * v)) + (be * g);
    if (a.r_g != 1.0) F = a.r_g * F;
    return F;
}

__global__ void k_step_f64(RefArgs a, int64_t q) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)a.N * a.R) return;
    int r = (int)(t / a.N), i = (int)(t % a.N);
    const double *x = a.phi_in + (int64_t)r * a.N;
    double F = ref_force(a, i, x, a.a64[2 * q], a.b64[2 * q]);
    double p = a.p[t];
    p = (q == 0) ? p - 0.5 * F : p - F;
    double ad = a.a64[2 * q + 1];
    if (a.r_g != 1.0) ad = a.r_g * ad;
    double xn = x[i] + (ad * p);
    a.p[t] = p;
    a.phi_out[t] = xn;
    if (q + 1 >= a.T - a.W + 1) a.S[t] = a.S[t] + xn;
    if (!isfinite(xn) || !isfinite(p)) atomicOr(a.err, ERR_NONFINITE);
}

static RefArgs ref_args(hqa_md *md, Instance &I) {
    RefArgs a;
    a.N = I.N; a.R = md->R; a.M = md->sch.M; a.csr = I.layout == HQA_CSR;
    a.T = md->sch.T; a.W = md->sch.W; a.r_g = md->sch.r_g;
    a.J = I.J64; a.rp = I.rp; a.ci = I.ci; a.h = I.h64;
    a.a64 = md->a64; a.b64 = md->b64;
    a.phi_in = nullptr; a.phi_out = nullptr; a.p = I.p64; a.S = I.S64; a.err = md->err;
    return a;
}

hipError_t launch_md_steps_f64(hqa_md *md, Instance &I, int64_t q0, int64_t q1) {
    RefArgs a = ref_args(md, I);
    int64_t n = (int64_t)I.N * md->R;
    unsigned blocks = (unsigned)((n + 255) / 256);
    for (int64_t q = q0; q < q1; q++) {
        a.phi_in = I.phi64[I.cur];
        a.phi_out = I.phi64[I.cur ^ 1];
        k_step_f64<<<blocks, 256, 0, md->stream>>>(a, q);
        I.cur ^= 1;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// binary64 field u = J phi from the binary64 couplings, for any state precision.
// ---------------------------------------------------------------------------
struct F64View {
    int N, R, ld, smaj, f64;
    const double *x64;
    const float *x32;
};

__device__ __forceinline__ double view_get(const F64View &v, int r, int i) {
    if (v.f64) return v.x64[(int64_t)r * v.N + i];
    int64_t k = v.smaj ? (int64_t)i * v.ld + r : (int64_t)r * v.ld + i;
    return (double)v.x32[k];
}

static F64View make_view(hqa_md *md, Instance &I, bool phi) {
    F64View v;
    v.N = I.N; v.R = md->R; v.ld = I.ld; v.smaj = I.smaj; v.f64 = md->prec == HQA_PREC_F64_REF;
    v.x64 = phi ? I.phi64[I.cur] : I.p64;
    v.x32 = phi ? I.phi32[I.cur] : I.p32;
    return v;
}

// One workgroup per replica: the replica's fluxes are staged in LDS in binary64.
__global__ void k_field_f64(RefArgs a, F64View xv, double *u) {
    extern __shared__ double xs[];
    int r = blockIdx.x;
    for (int i = threadIdx.x; i < a.N; i += blockDim.x) xs[i] = view_get(xv, r, i);
    __syncthreads();
    for (int i = threadIdx.x; i < a.N; i += blockDim.x) u[(int64_t)r * a.N + i] = ref_field(a, i, xs);
}

hipError_t launch_field_f64(hqa_md *md, Instance &I, double *u, hipStream_t st) {
    RefArgs a = ref_args(md, I);
    F64View xv = make_view(md, I, true);
    const size_t lds = (size_t)I.N * sizeof(double);   // one replica's fluxes in binary64
    hipError_t e = hipFuncSetAttribute((const void *)k_field_f64,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    k_field_f64<<<md->R, 256, lds, st>>>(a, xv, u);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// MD Hamiltonian (Eq. 3) at integer step q, binary64.
// The momentum at integer time is p^(q) = p^(q-1/2) - F(phi^(q))/2 (q >= 1).
// ---------------------------------------------------------------------------
struct HmdTerms {
    double kin, cpl, fld;
};

// The three sums' terms of one (spin, replica) with field u = (J phi)_i.
__device__ __forceinline__ HmdTerms hmd_terms(const RefArgs &a, int i, double x, double p, double u,
                                              double al, double be, int64_t q) {
    const double h = a.h[i];
    if (q > 0) {
        double v = x;
        for (int k = 0; k < a.M - 2; k++) v = v * x;
        const double g = u + (2.0 * h) * fabs(x);
        double F = (al * ((double)a.M * v)) + (be * g);
        if (a.r_g != 1.0) F = a.r_g * F;
        p = p - 0.5 * F;
    }
    double xm = x;
    for (int k = 0; k < a.M - 1; k++) xm = xm * x;
    return HmdTerms{0.5 * p * p + xm, x * u, h * fabs(x) * x};
}

// Sparse instances: one workgroup per replica, its fluxes staged in LDS.
__global__ void k_hamiltonian(RefArgs a, F64View xv, F64View pv, int64_t q, double *H) {
    extern __shared__ double xs[];
    __shared__ double red[3][256];
    int r = blockIdx.x;
    for (int i = threadIdx.x; i < a.N; i += blockDim.x) xs[i] = view_get(xv, r, i);
    __syncthreads();
    double al = a.a64[2 * q], be = a.b64[2 * q];
    double kin = 0.0, cpl = 0.0, fld = 0.0;
    for (int i = threadIdx.x; i < a.N; i += blockDim.x) {
        const HmdTerms t = hmd_terms(a, i, xs[i], view_get(pv, r, i), ref_field(a, i, xs), al, be, q);
        kin += t.kin;
        cpl += t.cpl;
        fld += t.fld;
    }
    red[0][threadIdx.x] = kin; red[1][threadIdx.x] = cpl; red[2][threadIdx.x] = fld;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int c = 0; c < 3; c++) red[c][threadIdx.x] += red[c][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) H[r] = al * red[0][0] + be * (0.5 * red[1][0] + red[2][0]);
}

// Dense instances: the field is a matrix product in binary64, bound by the 8 N^2 bytes of
// J, which are read once per 16 NT replicas.  A workgroup owns 16 rows x 16 NT replicas;
// its four wavefronts split the columns in contiguous quarters (16 columns a chunk) and
// run 16x16x4 binary64 MFMAs.  Within a chunk the lane group g = lane / 16 takes columns
// 4 g .. 4 g + 3, so that each lane reads 32 consecutive bytes of its row of J and 16 or
// 32 of its replica: MFMA v contracts columns {4 g + v}, the same for both operands, and
// the order of a binary64 sum is free here.  The quarters meet in LDS and the tile's terms
// are summed to one partial per (row tile, replica), added up in order by k_hmd_sum.
// Measured at N = 10^4, R = 16 (800 MB of J): 48.9 ms with one workgroup per replica and a
// thread per row (a row's doubles are read one per lane and line, and twice), 0.179 ms with this
// kernel (4.5 TB/s).
typedef double f64x2_u __attribute__((ext_vector_type(2), aligned(8)));
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

template <int NT, bool F64>
__global__ __launch_bounds__(256) void k_hmd_dense(RefArgs a, F64View xv, F64View pv, int64_t q,
                                                   double *part) {
    __shared__ double red[4][NT][256];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, kg = lane >> 4, l16 = lane & 15;
    const int N = a.N, i0 = blockIdx.y * 16, r0 = blockIdx.x * 16 * NT;
    // rows and replicas past the end repeat the last one; their results are not used
    const double *Jr = a.J + (int64_t)min(i0 + l16, N - 1) * N;
    int64_t xrow[NT];
#pragma unroll
    for (int t = 0; t < NT; t++)
        xrow[t] = (int64_t)min(r0 + 16 * t + l16, a.R - 1) * (F64 ? N : xv.ld);
    f64x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) acc[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    const int nfull = N / 16, nch = (N + 15) / 16, per = (nch + 3) / 4;
    const int c0 = w * per, c1 = min(nch, c0 + per);
#pragma unroll 4
    for (int c = c0; c < min(c1, nfull); c++) {
        const int k = 16 * c + 4 * kg;
        const f64x2_u j0 = *(const f64x2_u *)(Jr + k), j1 = *(const f64x2_u *)(Jr + k + 2);
        double x[NT][4];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if constexpr (F64) {
                const f64x2_u x0 = *(const f64x2_u *)(xv.x64 + xrow[t] + k);
                const f64x2_u x1 = *(const f64x2_u *)(xv.x64 + xrow[t] + k + 2);
                x[t][0] = x0[0]; x[t][1] = x0[1]; x[t][2] = x1[0]; x[t][3] = x1[1];
            } else {
                const float4 v = *(const float4 *)(xv.x32 + xrow[t] + k);   // ld is a multiple of 128
                x[t][0] = v.x; x[t][1] = v.y; x[t][2] = v.z; x[t][3] = v.w;
            }
        }
#pragma unroll
        for (int t = 0; t < NT; t++) {
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j0[0], x[t][0], acc[t], 0, 0, 0);
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j0[1], x[t][1], acc[t], 0, 0, 0);
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j1[0], x[t][2], acc[t], 0, 0, 0);
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j1[1], x[t][3], acc[t], 0, 0, 0);
        }
    }
    if (c0 <= nfull && nfull < c1 && nfull < nch) {   // the last, partial chunk
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int k = 16 * nfull + 4 * kg + v;
            const double j = k < N ? Jr[k] : 0.0;
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const double x = k < N ? (F64 ? xv.x64[xrow[t] + k] : (double)xv.x32[xrow[t] + k]) : 0.0;
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(j, x, acc[t], 0, 0, 0);
            }
        }
    }
    // accumulator v of a lane: row kg + 4 v, replica l16
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int v = 0; v < 4; v++) red[w][t][(kg + 4 * v) * 16 + l16] = acc[t][v];
    __syncthreads();
    const double al = a.a64[2 * q], be = a.b64[2 * q];
    const int i = i0 + (tid >> 4);
    HmdTerms s[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        const int r = r0 + 16 * t + (tid & 15);
        const double u = (red[0][t][tid] + red[1][t][tid]) + (red[2][t][tid] + red[3][t][tid]);
        s[t] = HmdTerms{0.0, 0.0, 0.0};
        if (i < N && r < a.R)
            s[t] = hmd_terms(a, i, view_get(xv, r, i), view_get(pv, r, i), u, al, be, q);
        for (int o = 16; o <= 32; o <<= 1) {   // the wavefront's four rows
            s[t].kin += __shfl_xor(s[t].kin, o);
            s[t].cpl += __shfl_xor(s[t].cpl, o);
            s[t].fld += __shfl_xor(s[t].fld, o);
        }
    }
    __syncthreads();
    if (lane < 16) {
#pragma unroll
        for (int t = 0; t < NT; t++) {
            red[w][t][l16] = s[t].kin;
            red[w][t][16 + l16] = s[t].cpl;
            red[w][t][32 + l16] = s[t].fld;
        }
    }
    __syncthreads();
    for (int e = tid; e < 48 * NT; e += 256) {
        const int t = e / 48, c = e % 48 / 16, r = r0 + 16 * t + (e & 15), k = 16 * c + (e & 15);
        if (r < a.R)
            part[((int64_t)blockIdx.y * 3 + c) * a.R + r] =
                (red[0][t][k] + red[1][t][k]) + (red[2][t][k] + red[3][t][k]);
    }
}

// H[r] from the row tiles' partial sums: one workgroup per replica.
__global__ __launch_bounds__(256) void k_hmd_sum(RefArgs a, int64_t q, int tiles, const double *part,
                                                 double *H) {
    __shared__ double red[3][4];
    const int r = blockIdx.x, tid = threadIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int t = tid; t < tiles; t += 256)
        for (int c = 0; c < 3; c++) s[c] += part[((int64_t)t * 3 + c) * a.R + r];
    for (int c = 0; c < 3; c++) {
        for (int o = 32; o > 0; o >>= 1) s[c] += __shfl_xor(s[c], o);
        if ((tid & 63) == 0) red[c][tid >> 6] = s[c];
    }
    __syncthreads();
    if (tid == 0) {
        for (int c = 0; c < 3; c++) s[c] = (red[c][0] + red[c][1]) + (red[c][2] + red[c][3]);
        H[r] = a.a64[2 * q] * s[0] + a.b64[2 * q] * (0.5 * s[1] + s[2]);
    }
}

// Bytes of device scratch launch_hamiltonian needs.
size_t hamiltonian_scratch_bytes(const Instance &I, int R) {
    return I.layout == HQA_DENSE ? (size_t)((I.N + 15) / 16) * 3 * R * sizeof(double) : 0;
}

template <int NT>
static void launch_hmd(const RefArgs &a, const F64View &xv, const F64View &pv, int64_t q,
                       double *part, hipStream_t st) {
    const dim3 grid((a.R + 16 * NT - 1) / (16 * NT), (a.N + 15) / 16);
    if (xv.f64) k_hmd_dense<NT, true><<<grid, 256, 0, st>>>(a, xv, pv, q, part);
    else k_hmd_dense<NT, false><<<grid, 256, 0, st>>>(a, xv, pv, q, part);
}

hipError_t launch_hamiltonian(hqa_md *md, Instance &I, double *H, void *scratch, hipStream_t st) {
    RefArgs a = ref_args(md, I);
    F64View xv = make_view(md, I, true), pv = make_view(md, I, false);
    if (!a.csr) {
        // J is read once per replica block: as wide a block as the replicas fill, while the blocks
        // give every CU one (whole call, wide / by this rule, R = 64: N = 8 32.9 / 30.7 us,
        // N = 500 39.0 / 32.9, N = 3000 84 / 76; R = 500: N = 8 35.8 / 32.9; a workgroup a replica
        // N = 8 29.1, 31.1, N = 500 105, 183)
        const int tiles = (a.N + 15) / 16;
        auto fills = [&](int reps) { return (int64_t)((a.R + reps - 1) / reps) * tiles >= 256; };
        if (a.R > 32 && fills(64)) launch_hmd<4>(a, xv, pv, md->q, (double *)scratch, st);
        else if (a.R > 16 && fills(32)) launch_hmd<2>(a, xv, pv, md->q, (double *)scratch, st);
        else launch_hmd<1>(a, xv, pv, md->q, (double *)scratch, st);
        k_hmd_sum<<<a.R, 256, 0, st>>>(a, md->q, (a.N + 15) / 16, (const double *)scratch, H);
        return hipGetLastError();
    }
    const size_t lds = (size_t)I.N * sizeof(double);
    hipError_t e = hipFuncSetAttribute((const void *)k_hamiltonian,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    k_hamiltonian<<<md->R, 256, lds, st>>>(a, xv, pv, md->q, H);
    return hipGetLastError();
}

}  // namespace hqa
