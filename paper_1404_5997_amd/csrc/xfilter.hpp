// Stride-1 filter gradient, fp32 storage, on the bf16 matrix unit with operands split in three (split3.hpp).
//
//   dw[k][r][s][c] = sum over (p,q) of  sum over images n of  dz[n,p,q,k] * x[n, p+r-pad_h, q+s-pad_w, c]
//
// (Section 4 of the paper, backward step 2.)  The inner sum is a matrix product whose reduction index is the image:
// a 16-deep matrix instruction takes 16 images at ONE output position.  That choice removes everything that made this
// pass awkward on NHWC data with the reduction over pixels:
//  * a lane's eight reduction values are eight images at the same position and channel, loaded by eight 4-byte loads
//    that are 128 consecutive bytes across a half-wavefront, split in registers and used as they are: no transposing
//    reads, no LDS, no barrier anywhere;
//  * a filter tap is the neighbouring position's fragment, unshifted.  Walking along an image row, the x fragment of a
//    position serves the S taps of a filter row one position after the other from a window of registers: it is loaded
//    and split once per row of taps;
//  * filter rows that fall outside the image are not computed at all (an r = 0 wavefront of a 13-high map walks over 12
//    output rows), and a row of 13 or 27 positions needs no rounding to chunks.
// A wavefront works alone: KB filter blocks of 32 x 32 channels x the S taps of one filter row, two accumulators each, one
// wavefront per SIMD with its 512 registers.  Work-groups of four of them hold neighbouring tiles of one split, so that
// what they load in common comes from one CU's cache.  The position range is split over wavefronts (partial sums in the
// workspace, splitk_reduce_kernel).
//
// What bounds it: the matrix instructions, as long as the vector instructions that split the next position's values
// issue in their shadow.  Measured with one wavefront per SIMD, a 32-cycle matrix instruction hides 28 cycles of vector
// issue, 5 cycles an instruction with a 4-byte encoding, 8 with an 8-byte one; a fragment's split is 256 cycles, so the
// KB + 1 fragments of a position cost 9 (KB = 2, 3 taps: of 36 instructions' 28) and 6 (KB = 1, 5 taps: of 30) times 28.
// Loads run one to two positions ahead, those of a row's start a whole row ahead.  The plain split has no test for values bf16
// cannot hold: infinite ones, or finite above the largest bf16, turn into NaN, which reaches every accumulator they touch, and
// those below 2^-110 lose bits, which only a result as small can show.  A wavefront whose sums are not all finite, or some
// below kSplitTiny and not zero, starts over with scaled operands and the careful split.
//
// TG = 4: layers whose positions do not fill the chip with long walks.  A wavefront's position is about 29 clocks a load instruction
// (16 to 24 of them), its splits and its products one after the other, so two wavefronts a SIMD (KB = 1, 3 taps) take less than twice
// as long; and four that share a tile need a quarter of the partial sums for the same length of walk, which were what limited the
// splits: 37 images 15x11, 100 -> 72, masked, 32.0 -> 23.4 us (42 splits of whole wavefronts, the fastest: 32.1); 16 images
// 14x14, 128 -> 128 26.7 -> 17.4; 4 of 28x28, 64 -> 64 26.0 -> 16.8.  170 drawn and odd layers, with xgather's: 7397 -> 5708 us,
// three of them more than 3 % slower (by 4 %).  At 128 images of 13x13 the two forms take the same (174 and 176).  KB = 2 (one wavefront a SIMD): 29 us
// on the first of these.
//
// Measured, 128 images, with the reduce pass, kernel on the fp32 instruction -> this one, us: 3x3 192->384 252 -> 151 (190
// TFLOP/s), 384->256 334 -> 191, 256->256 228 -> 137; 5x5 64->192 450 -> 271 (212 TFLOP/s).  Four wavefronts to a
// work-group instead of one: 149, 188, - and 266.
#pragma once
#include <type_traits>

#include "igemm.hpp"
#include "owt_host.hpp"
#include "split3.hpp"

namespace owt {

// (split, tile) pairs, split-major, four consecutive ones to the wavefronts of a work-group; the work-groups are dealt to
// the XCDs as owt_split_major_wg does.  Returns false for wavefronts past the last pair (there are no barriers).
__host__ __device__ inline int owt_split_major_wave_grid(int tiles, int splits) { return 8 * (((tiles * splits + 3) / 4 + 7) / 8); }
__device__ __forceinline__ bool owt_split_major_wave(int ntiles, int splits, int &tile, int &split)
{
    const int total = ntiles * splits, wgs = (total + 3) >> 2, xcd = blockIdx.x & 7, jx = blockIdx.x >> 3;
    if (jx >= (wgs >> 3) + (xcd < (wgs & 7) ? 1 : 0)) return false;
    const int pair = (xcd * (wgs >> 3) + min(xcd, wgs & 7) + jx) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (pair >= total) return false;
    split = pair / ntiles;
    tile = pair - split * ntiles;
    return true;
}

template <int KB, int S, int TG, bool MASKED>
__global__ void __launch_bounds__(256, xfilter_occ(KB, S, TG)) xfilter_kernel(const GemmParams p)
{
    constexpr int M = 6 * KB * S;                  // matrix instructions per position

    const Geom &g = p.g;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, split;
    if (TG > 1 ? !owt_split_major_wg(p.tiles_m * p.tiles_n, p.splits, tile, split) : !owt_split_major_wave(p.tiles_m * p.tiles_n, p.splits, tile, split)) return;
    const int kt = tile / p.tiles_n, rem = tile - kt * p.tiles_n;
    const int r = rem / p.ctiles, ct = rem - r * p.ctiles;
    const int k0 = kt * 32 * KB, c0 = ct * 32;

    // output rows whose input row p + r - pad_h exists, and this wavefront's range of (image group, row, column)
    const int p_lo = max(0, g.ph - r), Pv = max(0, min(g.P, g.H + g.ph - r) - p_lo), Q = g.Q;
    const int groups = (g.N + 15) >> 4, total = groups * Pv * Q;
    const int per = (total + p.splits - 1) / p.splits;
    const int g_beg = min(total, split * per), g_end = min(total, g_beg + per), sub = (per + TG - 1) / TG;
    const int o_beg = TG > 1 ? min(g_end, g_beg + wave * sub) : g_beg, o_end = TG > 1 ? min(g_end, o_beg + sub) : g_end;

    const unsigned imgx = (unsigned)(g.H * g.W * g.C) * 4u, imgz = (unsigned)(g.P * Q * g.K) * 4u;
    const unsigned xall = imgx * (unsigned)g.N, zall = imgz * (unsigned)g.N;
    // Byte offsets of a lane's eight images.  Images past the last are past the descriptor and read as zeros (the host has
    // checked that no offset of a group of 16 wraps round); channels and
    // filters past a ragged tile read whatever is there (inside the tensor, or zeros past its end) and only reach
    // accumulator rows and columns that are never stored.
    unsigned xo[8], zo[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        xo[j] = (unsigned)(8 * lh + j) * imgx + (unsigned)(c0 + li) * 4u;
        zo[j] = (unsigned)(8 * lh + j) * imgz + (unsigned)(k0 + li) * 4u;
    }

    split_acc big[KB][S], small[KB][S];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int s = 0; s < S; s++)
#pragma unroll
                for (int e = 0; e < 16; e++) big[kb][s][e] = small[kb][s][e] = 0.f;
    };
    float db[KB];
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] = 0.f;

    float sx = 1.f, sz = 1.f;                       // scales of x and dz in a careful run
    // DB: also sum dz over the positions (bias gradient).  CAREFUL: the second run, splits test for large values.
    auto walk = [&](auto db_tag, auto careful_tag) __attribute__((always_inline)) {
        constexpr bool DB = decltype(db_tag)::value, CAREFUL = decltype(careful_tag)::value;
        if (o_beg >= o_end) return;
        const unsigned xstep = (unsigned)g.C * 4u, zstep = (unsigned)g.K * 4u;
        // a row of the walk: byte offsets of its column 0 in x and in dz (image n0), its output columns [qa, qa + len)
        struct Row { unsigned x, z; int qa, len; };
        int left = o_end - o_beg, n0, prow, qa;
        {
            const int grp = o_beg / (Pv * Q), o = o_beg - grp * (Pv * Q);
            n0 = 16 * grp; prow = o / Q; qa = o - prow * Q;
        }
        auto next_row = [&]() __attribute__((always_inline)) {
            Row row;
            row.x = (unsigned)n0 * imgx + (unsigned)((prow + p_lo + r - g.ph) * g.W) * xstep;
            row.z = (unsigned)n0 * imgz + (unsigned)((prow + p_lo) * Q) * zstep;
            row.qa = qa;
            row.len = min(Q - qa, left);             // 0 past the end of the walk
            left -= row.len;
            qa = 0;
            if (++prow == Pv) { prow = 0; n0 += 16; }
            return row;
        };
        // x column qa - pad_w + i, output column qa + i of a row: zeros where there is none
        auto load_x = [&](const Row &row, int i, float (&v)[8]) __attribute__((always_inline)) {
            const int w = row.qa - g.pw + i;
            const __amdgpu_buffer_rsrc_t rs = owt_make_rsrc(p.b, row.len > 0 && (unsigned)w < (unsigned)g.W ? xall : 0u);
            const unsigned off = row.x + (unsigned)w * xstep;
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)xo[e], (int)off, 0));
        };
        auto load_z = [&](const Row &row, int i, int kb, float (&v)[8], float (&y)[8]) __attribute__((always_inline)) {
            const unsigned bytes = i < row.len ? zall : 0u, off = row.z + (unsigned)(row.qa + i) * zstep;
            const __amdgpu_buffer_rsrc_t rs = owt_make_rsrc(p.a, bytes);
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)zo[e] + kb * 128, (int)off, 0));
            if (MASKED) {
                const __amdgpu_buffer_rsrc_t ms = owt_make_rsrc(p.mask, bytes);
#pragma unroll
                for (int e = 0; e < 8; e++) y[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ms, (int)zo[e] + kb * 128, (int)off, 0));
            }
        };
        auto split = [&](const float (&v)[8], float scale, split_frag (&f)[3]) __attribute__((always_inline)) {
            if constexpr (CAREFUL) {
                float u[8];
#pragma unroll
                for (int e = 0; e < 8; e++) u[e] = v[e] * scale;
                split3_careful(u, f);
            } else {
                split3_plain(v, f);
            }
        };
        float row_db[KB];                            // the bias gradient's sum of a row: one long chain of additions rounds more
#pragma unroll
        for (int kb = 0; kb < KB; kb++) row_db[kb] = 0.f;
        auto split_z = [&](int kb, float (&v)[8], const float (&y)[8], split_frag (&f)[3]) __attribute__((always_inline)) {
            if (MASKED) {
#pragma unroll
                for (int e = 0; e < 8; e++) v[e] = y[e] > 0.f ? v[e] : 0.f;
            }
            if (DB) row_db[kb] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            split(v, sz, f);
        };

        // win[0..S-1]: x fragments of the S columns this position's taps meet; win[S]: the next column's, being split.
        // xf, zf: the first columns and the first position of the row ahead; xr, zr: of the position ahead.
        split_frag win[S + 1][3], az[KB][3];
        float xf[S][8], zf[KB][8], yf[MASKED ? KB : 1][8], xr[8], zr[KB][8], yr[MASKED ? KB : 1][8];
        Row row = next_row();
        auto load_first = [&](const Row &rw) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < S; i++) load_x(rw, i, xf[i]);
#pragma unroll
            for (int kb = 0; kb < KB; kb++) load_z(rw, 0, kb, zf[kb], yf[MASKED ? kb : 0]);
        };
        auto load_next = [&](const Row &rw, int i) __attribute__((always_inline)) {
            load_x(rw, i + S - 1, xr);
#pragma unroll
            for (int kb = 0; kb < KB; kb++) load_z(rw, i, kb, zr[kb], yr[MASKED ? kb : 0]);
        };
        load_first(row);
        load_next(row, 1);
        while (row.len > 0) {
            // (columns left of the image are zeros already: nothing to split)
#pragma unroll
            for (int i = 0; i < S; i++) {
                if (i < S - 1 && row.qa - g.pw + i < 0) {
#pragma unroll
                    for (int e = 0; e < 3; e++) win[i][e] = __builtin_bit_cast(split_frag, make_uint4(0u, 0u, 0u, 0u));
                } else {
                    split(xf[i], sx, win[i]);
                }
            }
#pragma unroll
            for (int kb = 0; kb < KB; kb++) split_z(kb, zf[kb], yf[MASKED ? kb : 0], az[kb]);
            const Row ahead = next_row();
            load_first(ahead);                       // a whole row's time to arrive
            for (int q = 0; q < row.len; q++) {
                // the products of position q, one phase per fragment of position q + 1: its vector instructions are spread
                // between the phase's matrix instructions, then its raw registers are loaded for position q + 2
                split_frag nz[KB][3];
                constexpr int PH = M / (KB + 1);
                const bool last = q + 2 > row.len;   // position q + 2 is then the second of the row ahead
                Row tgt = row;
                int ti = q + 2;
                if (last) { tgt = ahead; ti = 1; }
#pragma unroll
                for (int f = 0; f <= KB; f++) {
                    if (f == 0) { split(xr, sx, win[S]); load_x(tgt, ti + S - 1, xr); }
                    else { split_z(f - 1, zr[f - 1], yr[MASKED ? f - 1 : 0], nz[f - 1]); load_z(tgt, ti, f - 1, zr[f - 1], yr[MASKED ? f - 1 : 0]); }
#pragma unroll
                    for (int i = f * PH; i < (f == KB ? M : (f + 1) * PH); i++) {
                        constexpr int PA[6] = {0, 2, 0, 1, 1, 0}, PB[6] = {0, 0, 2, 1, 0, 1};
                        const int kb = i / (6 * S), e = i / S % 6, s = i % S;
                        split_acc &acc = e == 0 ? big[kb][s] : small[kb][s];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(az[kb][PA[e]], win[s][PB[e]], acc, 0, 0, 0);
                    }
                    constexpr int VPM = (44 + (MASKED ? 16 : 0) + (DB ? 8 : 0) + PH - 1) / PH;
#pragma unroll
                    for (int i = 0; i < PH; i++) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // a matrix instruction
                        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);     // vector instructions in its shadow
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int s = 0; s < S; s++)
#pragma unroll
                    for (int e = 0; e < 3; e++) win[s][e] = win[s + 1][e];
#pragma unroll
                for (int kb = 0; kb < KB; kb++)
#pragma unroll
                    for (int e = 0; e < 3; e++) az[kb][e] = nz[kb][e];
            }
            if (DB) {
#pragma unroll
                for (int kb = 0; kb < KB; kb++) { db[kb] += row_db[kb]; row_db[kb] = 0.f; }
            }
            row = ahead;
        }
    };

    clear();
    const bool do_db = ct == 0 && r == g.ph && p.dbias != nullptr;        // every output row has an input row there
    if (do_db) walk(std::true_type{}, std::false_type{});
    else walk(std::false_type{}, std::false_type{});
    // Is every sum finite, and none but zero so small that operands may have lost bits?  If not, once more with the split that
    // tests for large values: scaled up, and where that is not finite (or the first run was not) with products that no finite
    // operands take out of the range.
    float unscale = 1.f;
    unsigned low;
    auto all_finite = [&]() __attribute__((always_inline)) {
        float sum = 0.f;
        low = ~0u;                                   // of twice the bits, less one: zero counts as large
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int s = 0; s < S; s++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const float v = big[kb][s][e] + small[kb][s][e];
                    sum += v;
                    low = min(low, (__float_as_uint(v) << 1) - 1u);
                }
        return __ballot(!(fabsf(sum) < __builtin_inff())) == 0;
    };
    bool finite = all_finite();
    if (!finite || __ballot(low < (__float_as_uint(kSplitTiny) << 1) - 1u) != 0) {
        bool up = finite;
        do {
            sx = up ? kSplitScale : 1.f;
            sz = up ? kSplitScale : kSplitDown;
            unscale = up ? kSplitUnscale : kSplitUndown;
            clear();
            walk(std::false_type{}, std::true_type{});
            finite = all_finite() || !up;
            up = false;
        } while (!finite);
    }

    // register e of lane (li, lh): filter 8*(e/4) + 4*lh + e%4 of its block, channel li
    const bool part = p.splits > 1;
    float *out = part ? p.partial + (size_t)split * p.M * p.Ncols : (float *)p.out;
    const int c = c0 + li, RS = g.R * S;
    auto store = [&](int kb, int s, int e, float v) __attribute__((always_inline)) {
        const int k = k0 + kb * 32 + 8 * (e / 4) + 4 * lh + e % 4;
        if (k >= g.K) return;
        const size_t o = ((size_t)k * RS + r * S + s) * g.C + c;
        if (part) out[o] = v;
        else out[o] = p.alpha * v + (p.beta != 0.f ? p.beta * out[o] : 0.f);
    };
    auto store_db = [&](int kb, float v) __attribute__((always_inline)) {
        const int k = k0 + kb * 32 + li;
        if (lh || k >= g.K) return;
        if (part) p.dbias_partial[(size_t)split * p.M + k] = v;
        else p.dbias[k] = p.alpha * v + (p.beta != 0.f ? p.beta * p.dbias[k] : 0.f);
    };
    if constexpr (TG == 1) {
        if (c < g.C) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int s = 0; s < S; s++)
#pragma unroll
                    for (int e = 0; e < 16; e++) store(kb, s, e, (big[kb][s][e] + small[kb][s][e]) * unscale);
        }
        if (do_db) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++) store_db(kb, db[kb] + __shfl_xor(db[kb], 32));
        }
    } else {
        // the wavefronts' sums, added in pairs
        constexpr int V = KB * S * 16;
        __shared__ float red[TG * (V + KB) * 64];
        float *mine = red + wave * (V + KB) * 64 + lane;
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int s = 0; s < S; s++)
#pragma unroll
                for (int e = 0; e < 16; e++) mine[((kb * S + s) * 16 + e) * 64] = (big[kb][s][e] + small[kb][s][e]) * unscale;
#pragma unroll
        for (int kb = 0; kb < KB; kb++) mine[(V + kb) * 64] = db[kb] + __shfl_xor(db[kb], 32);
        __syncthreads();
        static_assert(TG == 4, "four wavefronts' sums in two pairs");
        for (int v = wave; v < V + KB; v += TG) {
            const float *at = red + v * 64 + lane;
            const float sum = (at[0] + at[(V + KB) * 64]) + (at[2 * (V + KB) * 64] + at[3 * (V + KB) * 64]);
            if (v >= V) { if (do_db) store_db(v - V, sum); }
            else if (c < g.C) store(v / (S * 16), v / 16 % S, v % 16, sum);
        }
    }
}

}  // namespace owt
