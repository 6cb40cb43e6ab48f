// The fully-connected column shard (Section 4 of the paper, forward step 3 / backward step 1), bf16 storage.
//
// xfc.hpp's decomposition (fragments straight from memory, the four wavefronts of a work-group share a 64 x 64 tile's reduction,
// one launch for both backward products) with loads laid out for 2-byte values: a 16-deep step of a wavefront is 128 clocks of matrix
// instructions, so what counts is how many loads it takes and how many of them are in flight.  Raw values stay packed (4 registers a
// fragment), which leaves room for the loads of three or four steps; an operand that is strided along the reduction is loaded two
// columns at a time, half as many loads.
// Measured, us, one step's loads in flight and 2-byte loads of columns -> here, forward and backward: 128 x 9216 -> 512
// 22.6, 20.9 -> 13.7, 20.2; 256 x 9216 -> 512 37.5, 35.5 -> 18.5, 30.4; 128 x 4096 -> 512 13.0, 13.5 -> 11.2, 10.8; 200 x 1024 -> 256 12.1, 8.7 -> 8.8, 7.4.
#pragma once
#include "igemm.hpp"
#include "split3.hpp"

namespace owt {

// One operand of a step: eight reduction values of this lane's row (or column) in each of the tile's two blocks of 32, raw.  ROW: the
// operand is contiguous along the reduction.  WIDE: 16-byte loads along a row, which ask for 4-byte aligned rows, or two
// neighbouring columns with one load (columns of block 0 are then the even ones of the tile); else one value a load.
template <bool ROW, bool WIDE> struct Xfc16Raw {
    static constexpr bool PAIR = !ROW && WIDE;
    static constexpr int NV = WIDE ? 8 : 16;
    uint32_t v[NV];

    // base: byte offset of the row (of block 0's column in row 0); len: values per stored row; k: this lane's first reduction index
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, unsigned base, unsigned len, int k)
    {
        if constexpr (ROW && WIDE) {
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const owt_u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(base + (unsigned)t * 64u * len + (unsigned)k * 2u), 0, 0);
                v[4 * t] = u.x; v[4 * t + 1] = u.y; v[4 * t + 2] = u.z; v[4 * t + 3] = u.w;
            }
        } else if constexpr (ROW) {
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int j = 0; j < 8; j++)
                    v[8 * t + j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)(base + (unsigned)t * 64u * len + (unsigned)(k + j) * 2u), 0, 0);
        } else {
            const unsigned at = base + (unsigned)k * len * 2u;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int off = (int)(at + (unsigned)j * len * 2u);
                if constexpr (WIDE) {
                    v[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
                } else {
                    v[j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
                    v[8 + j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off + 64, 0, 0);
                }
            }
        }
    }
    __device__ __forceinline__ uint4 words(int t) const            // block t's eight values
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if constexpr (ROW && WIDE) w[i] = v[4 * t + i];
            else if constexpr (WIDE) w[i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], t ? 0x07060302u : 0x05040100u);
            else w[i] = __builtin_amdgcn_perm(v[8 * t + 2 * i + 1], v[8 * t + 2 * i], 0x05040100u);
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};

// place in the tile of row (column) i of block t
template <bool PAIR> __device__ __forceinline__ int xfc16_place(int t, int i) { return PAIR ? 2 * i + t : 32 * t + i; }

// Block t of an operand as a fragment: masked by y > 0 (MASKED), zero at and past the reduction's end (`left` values of this lane's
// eight are left; 8 or more: all), summed up in `sum` (DB).
template <bool MASKED, bool DB, class Raw>
__device__ __forceinline__ split_frag xfc16_pack(const Raw &r, const Raw &y, int t, int left, float &sum)
{
    uint4 w = r.words(t);
    if (MASKED) w = mask_words16(w, y.words(t));
    if (left < 8) {
        auto keep = [&](int i) { return left >= 2 * i + 2 ? 0xffffffffu : (left == 2 * i + 1 ? 0xffffu : 0u); };
        w.x &= keep(0); w.y &= keep(1); w.z &= keep(2); w.w &= keep(3);
    }
    if (DB) sum += sum8_bf16(w);
    return __builtin_bit_cast(split_frag, w);
}

// A 64 x 64 tile of one product by one wavefront: reduction steps step0, step0 + stride, ... below nsteps (16 deep each), added to
// acc.  AROW / BROW: the operand is contiguous along the reduction.  Rows (A) and columns (B) past the end read harmlessly.
template <bool AROW, bool BROW, bool AWIDE, bool BWIDE, bool MASKED, bool DB>
__device__ __forceinline__ void xfc16_tile(const void *a, const void *y, const void *b, unsigned a_bytes, unsigned b_bytes, int a_len, int b_len, int Kd,
                                           int m0, int n0, int step0, int stride, int nsteps, split_acc (&acc)[2][2], float (&db)[2])
{
    typedef Xfc16Raw<AROW, AWIDE> RA;
    typedef Xfc16Raw<BROW, BWIDE> RB;
    constexpr int AHEAD = AWIDE && BWIDE ? (MASKED ? 3 : 4) : 2;     // steps whose loads are in flight: what two wavefronts a SIMD hold
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(a, a_bytes), brs = owt_make_rsrc(b, b_bytes);
    const __amdgpu_buffer_rsrc_t yrs = owt_make_rsrc(MASKED ? y : a, a_bytes);
    // byte offset of this lane's row (contiguous operand) or column (strided one) of block 0; *_len = values per stored row
    const unsigned ao = AROW ? (unsigned)(m0 + li) * (unsigned)a_len * 2u : (unsigned)(m0 + xfc16_place<RA::PAIR>(0, li)) * 2u;
    const unsigned bo = BROW ? (unsigned)(n0 + li) * (unsigned)b_len * 2u : (unsigned)(n0 + xfc16_place<RB::PAIR>(0, li)) * 2u;
    RA ra[AHEAD], ry[MASKED ? AHEAD : 1];
    RB rb[AHEAD];
    auto load = [&](int step, int u) __attribute__((always_inline)) {
        if (step >= nsteps) return;
        const int k = step * 16 + 8 * lh;
        ra[u].load(ars, ao, (unsigned)a_len, k);
        if (MASKED) ry[MASKED ? u : 0].load(yrs, ao, (unsigned)a_len, k);
        rb[u].load(brs, bo, (unsigned)b_len, k);
    };
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
#pragma unroll
    for (int u = 0; u < AHEAD; u++) load(step0 + u * stride, u);
    for (int s0 = step0; s0 < nsteps; s0 += AHEAD * stride) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            const int step = s0 + u * stride;
            if (step >= nsteps) break;
            const int left = step * 16 + 16 > Kd ? Kd - (step * 16 + 8 * lh) : 8;      // below 8 in the last step of a ragged reduction
            split_frag fa[2], fb[2];
            float none = 0.f;
#pragma unroll
            for (int t = 0; t < 2; t++) fa[t] = xfc16_pack<MASKED, DB>(ra[u], ry[MASKED ? u : 0], t, left, db[t]);
#pragma unroll
            for (int t = 0; t < 2; t++) fb[t] = xfc16_pack<false, false>(rb[u], rb[u], t, left, none);
            load(step + AHEAD * stride, u);
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }
}

// The four wavefronts' sums of one tile added in a fixed order; `store(row, column, value)` gets each value of the tile once.
template <bool APAIR, bool BPAIR, class Store>
__device__ __forceinline__ void xfc16_combine(float *red, const split_acc (&acc)[2][2], Store store)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++)
                red[wave * 4096 + xfc16_place<APAIR>(i, 8 * (e / 4) + 4 * lh + e % 4) * 64 + xfc16_place<BPAIR>(j, li)] = acc[i][j][e];
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < 16; q++) {
        const int at = q * 256 + tid;
        store(at >> 6, at & 63, (red[4096 + at] + red[at]) + (red[12288 + at] + red[8192 + at]));
    }
}

// EVEN: an even number of reduction values
template <bool EVEN>
__global__ void __launch_bounds__(256, 2) xfc16_fwd_kernel(const GemmParams p)
{
    __shared__ float red[4 * 4096];
    typedef EpiFwd<bf16_t> Epi;
    const int tn = blockIdx.x % p.tiles_n, tm = blockIdx.x / p.tiles_n, split = blockIdx.y, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = tm * 64, n0 = tn * 64, I = p.Kd;
    const int beg = split * p.ksteps_per_split, end = min(p.ksteps, beg + p.ksteps_per_split);
    split_acc acc[2][2];
    float db[2];
    xfc16_tile<true, true, EVEN, EVEN, false, false>(p.a, nullptr, p.b, (unsigned)p.M * I * 2u, (unsigned)p.Ncols * I * 2u, I, I, I, m0, n0, beg + wave, 4, end, acc, db);
    xfc16_combine<false, false>(red, acc, [&](int r, int c, float v) {
        const int m = m0 + r, n = n0 + c;
        if (m >= p.M || n >= p.Ncols) return;
        if (p.splits > 1) p.partial[((size_t)split * p.M + m) * p.Ncols + n] = v;
        else store1((bf16_t *)p.out, (size_t)m * p.Ncols + n, Epi::op(p, m, n, v));
    });
}

// Work-groups below pd.tiles_m * pd.tiles_n: a tile of dx; the others: a tile of dw.  Either range may be empty.  OE / IE: O and I
// are even.
template <bool MASKED, bool OE, bool IE>
__global__ void __launch_bounds__(256, 2) xfc16_bwd_kernel(const GemmParams pd, const GemmParams pf)
{
    __shared__ float red[4 * 4096];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ndx = pd.tiles_m * pd.tiles_n;
    const int N = pf.Kd, O = pf.M, I = pf.Ncols;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
    split_acc acc[2][2];
    float db[2] = {0.f, 0.f};
    if ((int)blockIdx.x < ndx) {
        const int tn = blockIdx.x % pd.tiles_n, tm = blockIdx.x / pd.tiles_n, m0 = tm * 64, n0 = tn * 64;
        xfc16_tile<true, false, OE, IE, MASKED, false>(pd.a, pd.mask, pd.b, (unsigned)N * O * 2u, (unsigned)O * I * 2u, O, I, O, m0, n0, wave, 4, (O + 15) >> 4, acc, db);
        xfc16_combine<false, IE>(red, acc, [&](int r, int c, float v) {
            const int m = m0 + r, n = n0 + c;
            if (m < N && n < I) store1((bf16_t *)pd.out, (size_t)m * I + n, EpiData<bf16_t>::op(pd, m, n, v));
        });
        return;
    }
    const int t = blockIdx.x - ndx, tm = t / pf.tiles_n, tn = t - tm * pf.tiles_n;
    const int m0 = tm * 64, n0 = tn * 64;
    const bool do_db = tn == 0 && pf.dbias != nullptr;
    const int nsteps = (N + 15) >> 4;
    if (do_db)
        xfc16_tile<false, false, OE, IE, MASKED, true>(pf.a, pf.mask, pf.b, (unsigned)N * O * 2u, (unsigned)N * I * 2u, O, I, N, m0, n0, wave, 4, nsteps, acc, db);
    else
        xfc16_tile<false, false, OE, IE, MASKED, false>(pf.a, pf.mask, pf.b, (unsigned)N * O * 2u, (unsigned)N * I * 2u, O, I, N, m0, n0, wave, 4, nsteps, acc, db);
    float *out = (float *)pf.out;
    xfc16_combine<OE, IE>(red, acc, [&](int r, int c, float v) {
        const int o = m0 + r, n = n0 + c;
        if (o >= O || n >= I) return;
        const size_t at = (size_t)o * I + n;
        out[at] = pf.alpha * v + (pf.beta != 0.f ? pf.beta * out[at] : 0.f);
    });
    if (do_db) {
        __syncthreads();                                         // everyone has read the tile's sums
#pragma unroll
        for (int i = 0; i < 2; i++) red[wave * 128 + lh * 64 + xfc16_place<OE>(i, li)] = db[i];
        __syncthreads();
        const int o = m0 + tid;
        if (tid < 64 && o < O) {
            float v = 0.f;
            for (int w = 0; w < 4; w++) v += red[w * 128 + tid] + red[w * 128 + 64 + tid];
            pf.dbias[o] = pf.alpha * v + (pf.beta != 0.f ? pf.beta * pf.dbias[o] : 0.f);
        }
    }
}

}  // namespace owt
