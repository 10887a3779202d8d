// k_md_csr.hip -- sparse field (CSR SpMM over replica-contiguous fluxes) with the
// leapfrog fused, one launch per MD step.
//
// Layout: the binary32 state is spin-major [N][Rp] (Rp = R padded to a multiple
// of 4): row i holds spin i of every replica, so a neighbour's fluxes are one
// contiguous run.  Per spin update the kernel moves 16 bytes of state (read phi,
// read and write p, write phi') and gathers 4 bytes per coupling.
#include "hqa_internal.h"
#include "md_epilogue.h"

namespace hqa {

struct CsrArgs {
    int N, R, Rq, M;     // Rq = Rp / 4 threads per row
    int64_t T;
    int W;
    float rg;
    const int32_t *rp, *ci;
    const float *v;
    const float *h;
    const float *a32, *b32;
    const float *phi_in;
    float *phi_out, *p, *S;
    float *u_out;
    int32_t *err;
    float *st;             // early-stop statistics (9 x state size) or null
    int64_t sst;           // stride between the nine statistics arrays
    const float *inv_n2;   // 1 / ||J_i||_2
};

template <int VEC>
using csr_vec = float __attribute__((ext_vector_type(VEC)));

// The update of VEC consecutive replicas of row i (at `base` in the state) with field u.
template <int VEC, bool FIELD_ONLY>
__device__ __forceinline__ void csr_update(const CsrArgs &a, int64_t q, int i, int64_t base,
                                           const csr_vec<VEC> &u, const csr_vec<VEC> &x, csr_vec<VEC> p) {
    typedef csr_vec<VEC> fv;
    if constexpr (FIELD_ONLY) {
        *(fv *)(a.u_out + base) = u;
        return;
    } else {
        const StepCoef cf = step_coef(a.a32, a.b32, q, a.rg, a.M);
        const float hi = a.h[i];
        fv xn;
        bool bad = false;
#pragma unroll
        for (int v = 0; v < VEC; v++) {
            float pv = p[v], nv;
            leapfrog(cf, x[v], u[v], hi, pv, nv);
            p[v] = pv;
            xn[v] = nv;
            bad |= !isfinite(nv) || !isfinite(pv);
        }
        if (a.st) {
            const float in2 = a.inv_n2[i];
#pragma unroll
            for (int v = 0; v < VEC; v++) es_accumulate(a.st, a.sst, base + v, x[v], xn[v], u[v], p[v], in2);
        }
        *(fv *)(a.phi_out + base) = xn;
        *(fv *)(a.p + base) = p;
        if (q + 1 >= a.T - a.W + 1) {
            fv s = *(const fv *)(a.S + base);
#pragma unroll
            for (int v = 0; v < VEC; v++) s[v] = s[v] + xn[v];
            *(fv *)(a.S + base) = s;
        }
        if (bad) atomicOr(a.err, ERR_NONFINITE);
    }
}

// One wavefront per (row, chunk of 64 VEC replicas), VEC consecutive replicas a lane; the
// row's couplings are walked in ascending column order.
//
// What bounds it is the gather's latency and then its bytes from L2, so
//  * the row is uniform over the wavefront: column indices and values come through scalar
//    loads, eight at a time, and a gather is one vector load with a 32-bit offset (O;
//    64-bit where the state reaches 4 GB);
//  * 16 (then 8) gathers are in flight together; the last batch reads the last coupling
//    again in place of those past the end and does not use it;
//  * workgroup b runs on XCD b mod 8, each XCD with its own L2.  Sliced, an XCD serves one
//    chunk of 64 replicas at a time (nchunk = 2, 4: 8 / nchunk XCDs split the rows of a
//    chunk; multiples of 8: chunks x, x + 8, ... on XCD x), so the fluxes an XCD gathers
//    from are 256 N bytes instead of all replicas'.  Otherwise each XCD has a contiguous
//    range of rows, whose neighbours are nearby in lattices.
//
// Measured, us per step (a thread per row and 4 replicas, one gather at a time -> now):
// G(10^4, mean degree 30) R = 16, 128, 512: 20.1, 24.8, 78.7 -> 7.6, 14.3, 42 (R = 128 is
// 154 MB of gathers, 13 TB/s from the L2s beyond the launch; unsliced 16.0);
// G(2000, 12) R = 128: 10.6 -> 4.6; the 16^3 lattice R = 128, 1024: 5.3, 16.9 -> 5.0, 16.7.
template <int VEC, bool FIELD_ONLY, typename O>
__global__ __launch_bounds__(256) void k_step_csr(CsrArgs a, int64_t q, uint32_t nchunk, int sliced) {
    typedef csr_vec<VEC> fv;
    typedef int32_t i32x8 __attribute__((ext_vector_type(8), aligned(4)));
    typedef float f32x8 __attribute__((ext_vector_type(8), aligned(4)));
    // read-only for the whole launch and uniform: scalar loads
    typedef const __attribute__((address_space(4))) int32_t cint;
    typedef const __attribute__((address_space(4))) float cfloat;
    typedef const __attribute__((address_space(4))) i32x8 cint8;
    typedef const __attribute__((address_space(4))) f32x8 cfloat8;
    const uint32_t nrb = ((uint32_t)a.N + 3) / 4, b = blockIdx.x, nb = gridDim.x;
    uint32_t rb, chunk;
    if (sliced) {
        const uint32_t xcd = b % 8, k = b / 8;
        if (nchunk < 8) {
            const uint32_t share = 8 / nchunk, per = (nrb + share - 1) / share;
            chunk = xcd / share;
            rb = (xcd % share) * per + k;
            if (k >= per) return;
        } else {
            chunk = xcd + 8 * (k / nrb);
            rb = k % nrb;
        }
    } else {
        // XCD x takes [x nb/8, (x+1) nb/8); the last nb mod 8 workgroups keep their index
        const uint32_t per = nb / 8, t = b < per * 8 ? (b % 8) * per + b / 8 : b;
        rb = t / nchunk;
        chunk = t % nchunk;
    }
    const int i = __builtin_amdgcn_readfirstlane((int)(rb * 4 + (threadIdx.x >> 6)));
    if (i >= a.N) return;
    const uint32_t Rp = 4u * (uint32_t)a.Rq, c = (chunk * 64 + (threadIdx.x & 63)) * VEC;
    if (c >= Rp) return;
    const cint *rp = (const cint *)a.rp, *ci = (const cint *)a.ci;
    const cfloat *wv = (const cfloat *)a.v;
    const O pitch = 4 * (O)Rp, off = 4 * (O)c;
    const char *X = (const char *)a.phi_in;
    const int64_t base = (int64_t)i * Rp + c;
    fv u = 0.f, x = 0.f, p = 0.f;
    if constexpr (!FIELD_ONLY) {
        x = *(const fv *)(a.phi_in + base);
        p = *(const fv *)(a.p + base);
    }
    const int e1 = rp[i + 1];   // up to 2^31 - 1: e is compared by its distance from it
    int e = rp[i];
    if constexpr (VEC <= 2) {   // four a lane: eight gathers are already 8 KB in flight
        for (; e1 - e >= 16; e += 16) {
            const i32x8 ja = *(cint8 *)(ci + e), jb = *(cint8 *)(ci + e + 8);
            const f32x8 wa = *(cfloat8 *)(wv + e), wb = *(cfloat8 *)(wv + e + 8);
            fv g[16];
#pragma unroll
            for (int k = 0; k < 8; k++) g[k] = *(const fv *)(X + ((O)ja[k] * pitch + off));
#pragma unroll
            for (int k = 0; k < 8; k++) g[8 + k] = *(const fv *)(X + ((O)jb[k] * pitch + off));
#pragma unroll
            for (int k = 0; k < 16; k++)
#pragma unroll
                for (int v = 0; v < VEC; v++) u[v] = fmaf(k < 8 ? wa[k & 7] : wb[k & 7], g[k][v], u[v]);
        }
    }
    for (; e1 - e >= 8; e += 8) {
        const i32x8 j = *(cint8 *)(ci + e);
        const f32x8 w = *(cfloat8 *)(wv + e);
        fv g[8];
#pragma unroll
        for (int k = 0; k < 8; k++) g[k] = *(const fv *)(X + ((O)j[k] * pitch + off));
#pragma unroll
        for (int k = 0; k < 8; k++)
#pragma unroll
            for (int v = 0; v < VEC; v++) u[v] = fmaf(w[k], g[k][v], u[v]);
    }
    const int left = e1 - e;
    if (left > 0) {
        fv g[8];
#pragma unroll
        for (int k = 0; k < 8; k++) g[k] = *(const fv *)(X + ((O)ci[e + min(k, left - 1)] * pitch + off));
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (k < left) {
#pragma unroll
                for (int v = 0; v < VEC; v++) u[v] = fmaf(wv[e + k], g[k][v], u[v]);
            }
    }
    csr_update<VEC, FIELD_ONLY>(a, q, i, base, u, x, p);
}

// A thread per (row, four replicas), rows side by side in a wavefront; column indices and values
// come through vector loads, and a row's couplings are walked in ascending column order with B
// gathers in flight.  The last batch reads the last coupling again in place of those past the end
// and does not use it.  Bound by the gathers' bytes and the state's: the 100^3 lattice, R = 64,
// 260 us a step, 1.0 GB of state at 4 TB/s and its gathers from L2 beside it.
template <int B, bool FIELD_ONLY, typename O>
__global__ __launch_bounds__(256) void k_step_csr_rows(CsrArgs a, int64_t q) {
    typedef csr_vec<4> fv;
    // workgroup b runs on XCD b mod 8: XCD x takes the threads' x-th eighth (the last nb mod 8
    // workgroups keep their index)
    const int64_t nb = gridDim.x, per = nb / 8, b = blockIdx.x;
    const int64_t t = (b < per * 8 ? (b % 8) * per + b / 8 : b) * 256 + threadIdx.x;
    if (t >= (int64_t)a.N * a.Rq) return;
    const int i = (int)(t / a.Rq), c4 = (int)(t - (int64_t)i * a.Rq);
    const int64_t base = 4 * t;
    const O pitch = 16 * (O)a.Rq, off = 16 * (O)c4;
    const char *X = (const char *)a.phi_in;
    fv u = 0.f, x = 0.f, p = 0.f;
    if constexpr (!FIELD_ONLY) {
        x = *(const fv *)(a.phi_in + base);
        p = *(const fv *)(a.p + base);
    }
    const int e1 = a.rp[i + 1];
    int e = a.rp[i];
    for (; e1 - e >= B; e += B) {
        fv g[B];
        float w[B];
#pragma unroll
        for (int k = 0; k < B; k++) {
            g[k] = *(const fv *)(X + ((O)a.ci[e + k] * pitch + off));
            w[k] = a.v[e + k];
        }
#pragma unroll
        for (int k = 0; k < B; k++)
#pragma unroll
            for (int v = 0; v < 4; v++) u[v] = fmaf(w[k], g[k][v], u[v]);
    }
    const int left = e1 - e;
    if (left > 0) {
        fv g[B - 1];
        float w[B - 1];
#pragma unroll
        for (int k = 0; k < B - 1; k++) {
            const int ek = e + min(k, left - 1);
            g[k] = *(const fv *)(X + ((O)a.ci[ek] * pitch + off));
            w[k] = a.v[ek];
        }
#pragma unroll
        for (int k = 0; k < B - 1; k++)
            if (k < left) {
#pragma unroll
                for (int v = 0; v < 4; v++) u[v] = fmaf(w[k], g[k][v], u[v]);
            }
    }
    csr_update<4, FIELD_ONLY>(a, q, i, base, u, x, p);
}

static CsrArgs csr_args(hqa_md *md, Instance &I) {
    CsrArgs a;
    a.N = I.N; a.R = md->R; a.Rq = I.Rp / 4; a.M = md->sch.M;
    a.T = md->sch.T; a.W = md->sch.W; a.rg = (float)md->sch.r_g;
    a.rp = I.rp; a.ci = I.ci; a.v = I.v32; a.h = I.h32; a.a32 = md->a32; a.b32 = md->b32;
    a.phi_in = I.phi32[I.cur]; a.phi_out = I.phi32[I.cur ^ 1];
    a.p = I.p32; a.S = I.S32; a.u_out = nullptr; a.err = md->err;
    a.st = nullptr; a.sst = (int64_t)I.N * I.ld; a.inv_n2 = I.inv_n2;
    return a;
}

template <int VEC, bool FO>
static void launch_vec(const CsrArgs &a, int64_t q, const CsrPlan &p, hipStream_t st) {
    const unsigned grid = (unsigned)csr_wave_blocks(a.N, p);
    if ((uint64_t)a.N * a.Rq * 16 < (1ull << 32))
        k_step_csr<VEC, FO, uint32_t><<<grid, 256, 0, st>>>(a, q, p.chunks, p.sliced);
    else
        k_step_csr<VEC, FO, uint64_t><<<grid, 256, 0, st>>>(a, q, p.chunks, p.sliced);
}

template <int B, bool FO>
static void launch_rows(const CsrArgs &a, int64_t q, hipStream_t st) {
    const unsigned grid = (unsigned)(((int64_t)a.N * a.Rq + 255) / 256);
    if ((uint64_t)a.N * a.Rq * 16 < (1ull << 32)) k_step_csr_rows<B, FO, uint32_t><<<grid, 256, 0, st>>>(a, q);
    else k_step_csr_rows<B, FO, uint64_t><<<grid, 256, 0, st>>>(a, q);
}

template <bool FO>
static void launch_csr(const CsrArgs &a, const Instance &I, int64_t q, hipStream_t st) {
    const CsrPlan p = csr_plan(a.N, I.nnz, I.max_deg, (uint32_t)I.Rp);
    if (p.rows == 2) launch_rows<2, FO>(a, q, st);
    else if (p.rows) launch_rows<6, FO>(a, q, st);
    else if (p.vec == 1) launch_vec<1, FO>(a, q, p, st);
    else if (p.vec == 2) launch_vec<2, FO>(a, q, p, st);
    else launch_vec<4, FO>(a, q, p, st);
}

hipError_t launch_md_steps_csr(hqa_md *md, Instance &I, int64_t q0, int64_t q1) {
    for (int64_t q = q0; q < q1; q++) {
        CsrArgs a = csr_args(md, I);
        if (I.st && stats_step(md, q)) a.st = I.st;
        launch_csr<false>(a, I, q, md->stream);
        I.cur ^= 1;
    }
    return hipGetLastError();
}

hipError_t launch_field_csr(hqa_md *md, Instance &I, float *u, hipStream_t st) {
    CsrArgs a = csr_args(md, I);
    a.u_out = u;
    launch_csr<true>(a, I, 0, st);
    return hipGetLastError();
}

}  // namespace hqa
