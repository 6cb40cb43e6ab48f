// Forward pass of the fully-connected column shard (Section 4 of the paper, forward step 3) in one launch, both storage types.
//
//   y[n][o] = sum_i x[n][i] w[o][i]
//
// xfc.hpp and xfc16.hpp split the reduction of a few 64 x 64 tiles over work-groups and add the parts up in a second launch, which costs
// a small shard as much as the products.  Here a tile is 16 x 16 (v_mfma_f32_16x16x32_bf16: a lane holds eight reduction values of one row,
// 32 bytes of it), so that 128 x 512 results are 256 work-groups; a work-group's sixteen wavefronts take every sixteenth step (32 deep in fp32,
// 64 in bf16) of the whole reduction and add up through LDS in a tree.  fp32 operands are split in three (split3.hpp) as in xfc.hpp, each
// by sixteen times as many work-groups, which long reductions feel.
// Measured, us, xfc and its reduce pass -> here: fp32 19 x 632 -> 193 10.5 -> 4.7, 172 x 376 -> 44 8.9 -> 4.6, 61 x 1792 -> 210 11.3 -> 8.7, but
// 128 x 9216 -> 512 20 and 38; bf16 252 x 1494 -> 123 8.9 -> 4.5, 9 x 439 -> 46 12.8 -> 5.8, 128 x 4096 -> 512 11.2 -> 10.2, but 128 x 9216 ->
// 512 13.7 and 18.7.  Forward and backward of 60 drawn shards 0.87 (fp32) and 0.84 (bf16) of the time before; error of y 0.97.  What bounds
// it: for small shards a launch and the latency of one chain of loads; for larger ones rows of w and x read once a tile, 10 TB/s
// from the L2 caches at 128 x 4096 -> 512 (eight wavefronts a work-group take the same).
#pragma once
#include "igemm.hpp"
#include "split3.hpp"
#include "xfc.hpp"

namespace owt {

typedef float owt_f32x4 __attribute__((ext_vector_type(4)));

// A step's reduction values of this lane, raw: 32 consecutive bytes of its row, so that a row's four lanes take a line of it
// (ODD: an odd number of reduction values in bf16, whose rows start at any 2 bytes: the aligned words around them, shifted into place).
template <class T, bool ODD> struct XfcsRaw;
template <bool ODD> struct XfcsRaw<bf16_t, ODD> {
    static constexpr int VALUES = 16;
    uint32_t v[ODD ? 9 : 8];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, unsigned off)
    {
        const unsigned at = ODD ? off & ~3u : off;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const owt_u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + 16u * h), 0, 0);
            v[4 * h] = u.x; v[4 * h + 1] = u.y; v[4 * h + 2] = u.z; v[4 * h + 3] = u.w;
        }
        if constexpr (ODD) v[8] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(at + 32u), 0, 0);
    }
    // shift: the row's offset inside its first word, in bits; left: values of this lane's that exist
    __device__ __forceinline__ void words(unsigned shift, int left, split_frag (&f)[2]) const
    {
        uint32_t w[8];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            w[i] = ODD ? __builtin_amdgcn_alignbit(v[ODD ? i + 1 : i], v[i], shift) : v[i];
            if (left < VALUES) w[i] &= left >= 2 * i + 2 ? 0xffffffffu : (left == 2 * i + 1 ? 0xffffu : 0u);
        }
#pragma unroll
        for (int h = 0; h < 2; h++) f[h] = __builtin_bit_cast(split_frag, make_uint4(w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]));
    }
};
template <> struct XfcsRaw<float, false> {
    static constexpr int VALUES = 8;
    XfcOps::Raw r;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, unsigned off) { XfcOps::load_row(rs, off, 0, r); }
    __device__ __forceinline__ void keep(int left) { XfcOps::keep(r, 0, left); }
};

// Steps step0, step0 + stride, ... of a 16 x 16 tile, AHEAD of them in flight: the sums of the high parts' products and of the others
// (bf16: of the two halves of a step).
template <class T, bool ODD, int AHEAD, bool CAREFUL>
__device__ __forceinline__ void xfcs_run(const GemmParams &p, int m0, int n0, int step0, int stride, owt_f32x4 &big, owt_f32x4 &small)
{
    typedef XfcsRaw<T, ODD> Raw;
    constexpr unsigned ES = sizeof(T), V = Raw::VALUES;
    constexpr int DEEP = 4 * V;
    const int lane = threadIdx.x & 63, r = lane & 15, I = p.Kd, nsteps = (I + DEEP - 1) / DEEP;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(p.a, ((unsigned)p.M * (unsigned)I * ES + 3u) & ~3u), brs = owt_make_rsrc(p.b, ((unsigned)p.Ncols * (unsigned)I * ES + 3u) & ~3u);
    const unsigned ao = ((unsigned)(m0 + r) * (unsigned)I + V * (lane >> 4)) * ES, bo = ((unsigned)(n0 + r) * (unsigned)I + V * (lane >> 4)) * ES;
    big = small = {0.f, 0.f, 0.f, 0.f};
    Raw ra[AHEAD], rb[AHEAD];
    auto load = [&](int step, int u) __attribute__((always_inline)) {
        if (step >= nsteps) return;
        ra[u].load(ars, ao + (unsigned)step * DEEP * ES);
        rb[u].load(brs, bo + (unsigned)step * DEEP * ES);
    };
#pragma unroll
    for (int u = 0; u < AHEAD; u++) load(step0 + u * stride, u);
    for (int s0 = step0; s0 < nsteps; s0 += AHEAD * stride) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            const int step = s0 + u * stride;
            if (step >= nsteps) break;
            // the last step of a ragged reduction: what lies past it belongs to the next row
            const int left = step * DEEP + DEEP > I ? I - (step * DEEP + (int)V * (lane >> 4)) : (int)V;
            if constexpr (ES == 2) {
                split_frag a[2], b[2];
                ra[u].words((ao & 2u) * 8u, left, a);
                rb[u].words((bo & 2u) * 8u, left, b);
                load(step + AHEAD * stride, u);
                big = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], big, 0, 0, 0);
                small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], small, 0, 0, 0);
            } else {
                if (left < (int)V) { ra[u].keep(left); rb[u].keep(left); }
                const XfcOps::Frag a = XfcOps::pack<CAREFUL>(ra[u].r, CAREFUL ? kSplitDown : kSplitScale), b = XfcOps::pack<CAREFUL>(rb[u].r, CAREFUL ? 1.f : kSplitScale);
                load(step + AHEAD * stride, u);
                big = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[0], big, 0, 0, 0);
                constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int q = 0; q < 5; q++) small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[PA[q]], b.p[PB[q]], small, 0, 0, 0);
            }
        }
    }
}

template <class T, bool ODD>
__global__ void __launch_bounds__(1024, 4) xfcs_fwd_kernel(const GemmParams p)
{
    typedef EpiFwd<T> Epi;
    constexpr int NW = 16, HALVES = sizeof(T) == 4 ? 2 : 1;
    __shared__ float red[HALVES * NW * 256];
    // the tiles of one XCD share rows of w: in runs along the columns of x's rows
    const int ntiles = p.tiles_m * p.tiles_n, b = blockIdx.x, xcd = b & 7;
    const int logical = xcd * (ntiles >> 3) + min(xcd, ntiles & 7) + (b >> 3);
    const int tn = logical / p.tiles_m, tm = logical - tn * p.tiles_m, m0 = tm * 16, n0 = tn * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int AHEAD = sizeof(T) == 2 ? 4 : 2;
    owt_f32x4 big, small;
    xfcs_run<T, ODD, AHEAD, false>(p, m0, n0, wave, NW, big, small);
    if constexpr (sizeof(T) == 2) {
        big += small;
    } else {
        // as in xfc.hpp: operands are scaled up, and a wavefront whose sums are not finite starts over
        const owt_f32x4 v = big + small;
        const float sum = (v.x + v.y) + (v.z + v.w);
        float scale = kSplitUnscale;
        if (__ballot(!(fabsf(sum) < __builtin_inff())) != 0) {
            xfcs_run<T, ODD, 1, true>(p, m0, n0, wave, NW, big, small);
            scale = kSplitUndown;
        }
        big *= scale;
        small *= scale;
    }
    // value q of lane l is row 4 * (l / 16) + q, column l % 16
#pragma unroll
    for (int q = 0; q < 4; q++) {
        red[wave * 256 + q * 64 + lane] = big[q];
        if (HALVES == 2) red[(NW + wave) * 256 + q * 64 + lane] = small[q];
    }
    __syncthreads();
    if (tid >= 256) return;
    float y = 0.f;                                               // (the high parts' products by themselves: nearly exact sums)
#pragma unroll
    for (int h = 0; h < HALVES; h++) {
        float s[NW];
#pragma unroll
        for (int w = 0; w < NW; w++) s[w] = red[(h * NW + w) * 256 + tid];
#pragma unroll
        for (int d = 1; d < NW; d *= 2)
#pragma unroll
            for (int w = 0; w < NW; w += 2 * d) s[w] += s[w + d];
        y = h ? y + s[0] : s[0];
    }
    const int m = m0 + 4 * (lane >> 4) + (tid >> 6), n = n0 + (lane & 15);
    if (m < p.M && n < p.Ncols) store1((T *)p.out, (size_t)m * p.Ncols + n, Epi::op(p, m, n, y));
}

}  // namespace owt
