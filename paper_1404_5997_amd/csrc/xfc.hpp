// The fully-connected column shard (Section 4 of the paper, forward step 3 / backward step 1), fp32 storage, on the bf16 matrix
// unit with operands split in three (split3.hpp).  xfc16.hpp is the same for bf16 storage.
//
//   forward    y[n][o]  = sum_i x[n][i] w[o][i]         both operands contiguous along the reduction
//   data       dx[n][i] = sum_o dz[n][o] w[o][i]        dz contiguous, w strided
//   filter     dw[o][i] = sum_n dz[n][o] x[n][i]        both strided
//
// At a batch of 128 these products are a few microseconds of matrix or memory time, so what counts is launches, latency
// and wavefronts in flight.  Operands go from global memory straight into registers as matrix fragments (a fragment lane
// holds eight reduction values of one row or column: 32 contiguous bytes, or eight 4-byte loads that are contiguous across
// lanes); no LDS staging, no padding, no barrier in the loop, any N, I, O: what lies past the reduction
// is zeroed in the last step, rows and columns past the result read something harmless and are not stored.  dz = dy * [y > 0]
// is formed on the way into the fragments and the bias gradient in the filter product's wavefronts, so a backward call
// is one launch for both products.
// The four wavefronts of a work-group take every fourth 16-deep step of the reduction on one 64 x 64 tile and add up through
// LDS in a fixed order; forward splits the reduction over work-groups, too (partial sums, splitk_reduce_kernel).  (A step
// takes a lone wavefront 1.7 us in fp32: loads, split and products one after the other.  A wavefront per tile of dw, the
// whole batch as its reduction: 34 us instead of 30 for the backward call of 128 x 9216 -> 512, 18.3 instead of 8.4 for
// 4096 -> 125.)
//
// Measured, 128 images, us, direct-to-LDS GEMM on the fp32 instruction and a launch for dz -> here: 9216 -> 512 forward 20.1 -> 18.4,
// backward 32.6 -> 29.8; 4096 -> 512 16.0 -> 13.2 and 22.6 -> 16.2; 4096 -> 125 10.6 -> 10.7 and 11.0 -> 8.4.  What bounds it is the chain of a
// step: about 210 vector instructions that split its 4 x 8 values, then 24 matrix instructions.  Four steps' loads in flight at
// one wavefront per SIMD: forward 20.5 -> 24.9, backward 33 -> 86 (664 spilled registers); two neighbouring columns with an 8-byte
// load: backward 33 -> 38.  The forward pass reads more than its operands, too: with the split in blockIdx.y the work-groups of a column tile
// come to one XCD, and each of the eight reads all of x (9216 -> 512: 57 MB, the operands are 24).
#pragma once
#include "igemm.hpp"
#include "split3.hpp"

namespace owt {

// Eight raw values of a lane, and the fragments made of them.
struct XfcOps {
    struct Frag { split_frag p[3]; };
    struct Raw { uint32_t v[8]; };

    // CAREFUL: the second run, with a test for large values
    template <bool CAREFUL> static __device__ __forceinline__ Frag pack(const Raw &r, float scale)
    {
        Frag f;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = __uint_as_float(r.v[j]) * scale;
        if constexpr (CAREFUL) split3_careful(v, f.p);
        else split3_plain(v, f.p);
        return f;
    }
    static __device__ __forceinline__ float value(uint32_t v) { return __uint_as_float(v); }

    // Reduction values k .. k+7 of a row that is contiguous along the reduction; base = the row's byte offset.
    static __device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t rs, unsigned base, int k, Raw &r)
    {
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const owt_u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(base + (unsigned)(k + 4 * q) * 4u), 0, 0);
            r.v[4 * q] = t.x; r.v[4 * q + 1] = t.y; r.v[4 * q + 2] = t.z; r.v[4 * q + 3] = t.w;
        }
    }
    // The same where consecutive reduction values are `pitch` bytes apart; base = the column's byte offset in row k.
    static __device__ __forceinline__ void load_col(__amdgpu_buffer_rsrc_t rs, unsigned base, unsigned pitch, Raw &r)
    {
#pragma unroll
        for (int j = 0; j < 8; j++) r.v[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(base + (unsigned)j * pitch), 0, 0);
    }
    static __device__ __forceinline__ void keep(Raw &r, int k, int end)     // zeroes values at and past the reduction's end
    {
#pragma unroll
        for (int j = 0; j < 8; j++) r.v[j] = k + j < end ? r.v[j] : 0u;
    }
    static __device__ __forceinline__ void mask(Raw &r, const Raw &y)       // dy * [y > 0]
    {
#pragma unroll
        for (int j = 0; j < 8; j++) r.v[j] = value(y.v[j]) > 0.f ? r.v[j] : 0u;
    }
};

__device__ __forceinline__ void xfc_clear(split_acc (&a)[2][2], split_acc (&b)[2][2])
{
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) a[i][j][e] = b[i][j][e] = 0.f;
}

// A 64 x 64 tile of one product by one wavefront: reduction steps step0, step0 + stride, ... below nsteps (16 deep each).
// AROW / BROW: the operand is contiguous along the reduction.  Rows (A) and columns (B) past the end read harmlessly.
template <bool AROW, bool BROW, bool MASKED, bool DB, bool CAREFUL>
__device__ __forceinline__ void xfc_tile_run(const void *a, const void *y, const void *b, unsigned a_bytes, unsigned b_bytes, int a_len,
                                         int b_len, int Kd, int m0, int n0, int step0, int stride, int nsteps,
                                         split_acc (&big)[2][2], split_acc (&small)[2][2], float (&db)[2])
{
    typedef XfcOps O;
    constexpr unsigned ES = 4;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(a, a_bytes), brs = owt_make_rsrc(b, b_bytes);
    const __amdgpu_buffer_rsrc_t yrs = owt_make_rsrc(MASKED ? y : a, a_bytes);
    // byte offset of this lane's row (contiguous operand) or column (strided one); *_len = values per stored row
    unsigned ao[2], bo[2];
#pragma unroll
    for (int t = 0; t < 2; t++) {
        ao[t] = AROW ? (unsigned)(m0 + t * 32 + li) * (unsigned)a_len * ES : (unsigned)(m0 + t * 32 + li) * ES;
        bo[t] = BROW ? (unsigned)(n0 + t * 32 + li) * (unsigned)b_len * ES : (unsigned)(n0 + t * 32 + li) * ES;
    }
    typename O::Raw ra[2], ry[2], rb[2];
    auto load = [&](int step) __attribute__((always_inline)) {
        const int k = step * 16 + 8 * lh;
#pragma unroll
        for (int t = 0; t < 2; t++) {
            if constexpr (AROW) {
                O::load_row(ars, ao[t], k, ra[t]);
                if (MASKED) O::load_row(yrs, ao[t], k, ry[t]);
            } else {
                O::load_col(ars, ao[t] + (unsigned)k * (unsigned)a_len * ES, (unsigned)a_len * ES, ra[t]);
                if (MASKED) O::load_col(yrs, ao[t] + (unsigned)k * (unsigned)a_len * ES, (unsigned)a_len * ES, ry[t]);
            }
            if constexpr (BROW) O::load_row(brs, bo[t], k, rb[t]);
            else O::load_col(brs, bo[t] + (unsigned)k * (unsigned)b_len * ES, (unsigned)b_len * ES, rb[t]);
        }
    };
    if (step0 < nsteps) load(step0);
    for (int step = step0; step < nsteps; step += stride) {
        const int k = step * 16 + 8 * lh;
        typename O::Frag fa[2], fb[2];
        if (step * 16 + 16 > Kd) {                               // the last step of a ragged reduction
#pragma unroll
            for (int t = 0; t < 2; t++) { O::keep(ra[t], k, Kd); O::keep(rb[t], k, Kd); }
        }
#pragma unroll
        for (int t = 0; t < 2; t++) {
            if (MASKED) O::mask(ra[t], ry[t]);
            if (DB) {
                const auto v = [&](int j) { return O::value(ra[t].v[j]); };
                db[t] += ((v(0) + v(1)) + (v(2) + v(3))) + ((v(4) + v(5)) + (v(6) + v(7)));
            }
            fa[t] = O::template pack<CAREFUL>(ra[t], CAREFUL ? kSplitDown : kSplitScale);
            fb[t] = O::template pack<CAREFUL>(rb[t], CAREFUL ? 1.f : kSplitScale);
        }
        if (step + stride < nsteps) load(step + stride);
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                big[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].p[0], fb[j].p[0], big[i][j], 0, 0, 0);
        constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
        for (int q = 0; q < 5; q++)
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++)
                    small[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].p[PA[q]], fb[j].p[PB[q]], small[i][j], 0, 0, 0);
    }
}

// The tile's sums in `big` (both to be cleared before) and what they are to be multiplied with: fp32 operands are scaled up, and
// a wavefront whose sums are not finite starts over with products that no finite operands take out of the range.
template <bool AROW, bool BROW, bool MASKED, bool DB>
__device__ __forceinline__ float xfc_tile(const void *a, const void *y, const void *b, unsigned a_bytes, unsigned b_bytes, int a_len,
                                         int b_len, int Kd, int m0, int n0, int step0, int stride, int nsteps,
                                         split_acc (&big)[2][2], split_acc (&small)[2][2], float (&db)[2])
{
    xfc_tile_run<AROW, BROW, MASKED, DB, false>(a, y, b, a_bytes, b_bytes, a_len, b_len, Kd, m0, n0, step0, stride, nsteps, big, small, db);
    auto add_up = [&]() __attribute__((always_inline)) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    big[i][j][e] += small[i][j][e];
                    sum += big[i][j][e];
                }
        return sum;
    };
    if (__ballot(!(fabsf(add_up()) < __builtin_inff())) == 0) return kSplitUnscale;
    xfc_clear(big, small);
    xfc_tile_run<AROW, BROW, MASKED, false, true>(a, y, b, a_bytes, b_bytes, a_len, b_len, Kd, m0, n0, step0, stride, nsteps, big, small, db);
    add_up();
    return kSplitUndown;
}

// The four wavefronts' sums of one tile, each times its `scale`, added in a fixed order; `store(row, column, value)` gets each
// value of the tile once.
constexpr int kXfcRed = 4 * 4096 + 4;
template <class Store>
__device__ __forceinline__ void xfc_combine(float *red, const split_acc (&big)[2][2], float scale, Store store)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++)
                red[wave * 4096 + (i * 32 + 8 * (e / 4) + 4 * lh + e % 4) * 64 + j * 32 + li] = big[i][j][e];
    if (lane == 0) red[4 * 4096 + wave] = scale;
    __syncthreads();
    float s[4];
#pragma unroll
    for (int w = 0; w < 4; w++) s[w] = red[4 * 4096 + w];
#pragma unroll 4
    for (int q = 0; q < 16; q++) {
        const int at = q * 256 + tid;
        store(at >> 6, at & 63, fmaf(red[4096 + at], s[1], red[at] * s[0]) + fmaf(red[12288 + at], s[3], red[8192 + at] * s[2]));
    }
}

template <class Epi>
__global__ void __launch_bounds__(256, 2) xfc_fwd_kernel(const GemmParams p)
{
    __shared__ float red[kXfcRed];
    typedef typename Epi::TOut T;
    const int tn = blockIdx.x % p.tiles_n, tm = blockIdx.x / p.tiles_n, split = blockIdx.y, wave = threadIdx.x >> 6;
    const int m0 = tm * 64, n0 = tn * 64, I = p.Kd;
    const int beg = split * p.ksteps_per_split, end = min(p.ksteps, beg + p.ksteps_per_split);
    split_acc big[2][2], small[2][2];
    float db[2];
    xfc_clear(big, small);
    const float scale = xfc_tile<true, true, false, false>(p.a, nullptr, p.b, (unsigned)p.M * I * 4u, (unsigned)p.Ncols * I * 4u, I, I,
                                           I, m0, n0, beg + wave, 4, end, big, small, db);
    xfc_combine(red, big, scale, [&](int r, int c, float v) {
        const int m = m0 + r, n = n0 + c;
        if (m >= p.M || n >= p.Ncols) return;
        if (p.splits > 1) p.partial[((size_t)split * p.M + m) * p.Ncols + n] = v;
        else store1((T *)p.out, (size_t)m * p.Ncols + n, Epi::op(p, m, n, v));
    });
}

// Work-groups below pd.tiles_m * pd.tiles_n: a tile of dx; the others: a tile of dw.  Either range may be empty.
template <bool MASKED>
__global__ void __launch_bounds__(256, 2) xfc_bwd_kernel(const GemmParams pd, const GemmParams pf)
{
    __shared__ float red[kXfcRed];
    typedef float T;
    constexpr unsigned ES = 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ndx = pd.tiles_m * pd.tiles_n;
    const int N = pf.Kd, O = pf.M, I = pf.Ncols;
    split_acc big[2][2], small[2][2];
    float db[2] = {0.f, 0.f};
    xfc_clear(big, small);
    if ((int)blockIdx.x < ndx) {
        const int tn = blockIdx.x % pd.tiles_n, tm = blockIdx.x / pd.tiles_n, m0 = tm * 64, n0 = tn * 64;
        const float scale = xfc_tile<true, false, MASKED, false>(pd.a, pd.mask, pd.b, (unsigned)N * O * ES, (unsigned)O * I * ES, O, I, O, m0, n0, wave, 4,
                                                 (O + 15) >> 4, big, small, db);
        xfc_combine(red, big, scale, [&](int r, int c, float v) {
            const int m = m0 + r, n = n0 + c;
            if (m < N && n < I) store1((T *)pd.out, (size_t)m * I + n, EpiData<T>::op(pd, m, n, v));
        });
        return;
    }
    const int t = blockIdx.x - ndx, tm = t / pf.tiles_n, tn = t - tm * pf.tiles_n;
    const int m0 = tm * 64, n0 = tn * 64, tid = threadIdx.x, lane = tid & 63;
    const bool do_db = tn == 0 && pf.dbias != nullptr;
    float scale;
    if (do_db)
        scale = xfc_tile<false, false, MASKED, true>(pf.a, pf.mask, pf.b, (unsigned)N * O * ES, (unsigned)N * I * ES, O, I, N, m0, n0, wave, 4,
                                                 (N + 15) >> 4, big, small, db);
    else
        scale = xfc_tile<false, false, MASKED, false>(pf.a, pf.mask, pf.b, (unsigned)N * O * ES, (unsigned)N * I * ES, O, I, N, m0, n0, wave, 4,
                                                  (N + 15) >> 4, big, small, db);
    float *out = (float *)pf.out;
    xfc_combine(red, big, scale, [&](int r, int c, float v) {
        const int o = m0 + r, n = n0 + c;
        if (o >= O || n >= I) return;
        const size_t at = (size_t)o * I + n;
        out[at] = pf.alpha * v + (pf.beta != 0.f ? pf.beta * out[at] : 0.f);
    });
    if (do_db) {
        __syncthreads();                                         // everyone has read the tile's sums
#pragma unroll
        for (int i = 0; i < 2; i++) red[wave * 128 + i * 64 + lane] = db[i];
        __syncthreads();
        const int o = m0 + tid;
        if (tid < 64 && o < O) {
            float v = 0.f;
            for (int w = 0; w < 4; w++) v += red[w * 128 + (tid >> 5) * 64 + (tid & 31)] + red[w * 128 + (tid >> 5) * 64 + 32 + (tid & 31)];
            pf.dbias[o] = pf.alpha * v + (pf.beta != 0.f ? pf.beta * pf.dbias[o] : 0.f);
        }
    }
}

}  // namespace owt
