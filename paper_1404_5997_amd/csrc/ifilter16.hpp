// Stride-1 filter gradient, bf16 storage, any channel counts, with the reduction over images.
//
//   dw[k][r][s][c] = sum over (p,q) of  sum over images n of  dz[n,p,q,k] * x[n, p+r-pad_h, q+s-pad_w, c]
//
// (Section 4 of the paper, backward step 2.)  As in xfilter.hpp a 16-deep matrix instruction takes 16 images at one output
// position: a lane's eight reduction values are eight images at the same position and channel, so operands are used as they
// are loaded, a filter tap is the neighbouring position's fragment, and there is no LDS, no barrier (but at the walk's end) and no
// condition on channel counts.  The kernels that stage pixels in LDS (dfilter_bf16.hpp, dfilter16b.hpp) move 16-byte pieces and are the
// faster ones where channel counts are multiples of eight and a chunk's rows fit their panel; this one takes the rest, which
// ran on the gather kernel with the fp32 instruction before.
//  * Where a tile is two blocks of 32 channels (or filters) and their number is even, a lane loads two neighbouring channels
//    of an image with one 4-byte load: columns of block 0 are the even channels of the tile, those of block 1 the odd ones.
//    Else a lane loads 2 bytes of its channel.  Loads are what bounds this kernel, so that is twice the rate.
//  * A wavefront walks over the columns of x under its output rows: column by column it loads x and, S - 1 columns behind,
//    dz.  Packed fragments of the last S columns stay in a ring of S + 1 (the next one is packed between the matrix
//    instructions of this one), raw loads run S + 1 columns ahead (half as many where
//    registers are short); the ring's places are compile-time constants of the
//    unrolled loop, so nothing is moved from register to register.
//
// What bounds it: a load instruction costs a wavefront 29 clocks, sixteen to forty of them a column against 96 to 384 clocks
// of matrix instructions, and where few wavefronts run the latency of loads, of which a wavefront can have 63 in flight.
// (Packing and loads spread between the matrix instructions: up to 250 registers spilled, 5 % slower where none were.)
//
// Four wavefronts of a work-group share a tile's positions and add their sums, in pairs, through LDS, a filter block by a channel block at
// a time.  With a tile to every wavefront the partial sums were four times as many for the same length of walk, and their stores and the reduce pass
// half of the time of layers that do not fill the chip: 127 layers that stayed with this kernel 9256 -> 8289 us, those under 30 us 0.78 of
// before, three more than 4 % slower (by 8 % at most), error of dw 0.97 of before on average; 10 images 39x6, 68 -> 64 of 5x5 24.0 -> 17.9,
// 126 of 37x38, 92 -> 191 of 5x5 366 -> 334.
//
// Measured with the reduce pass, a tile to a wavefront, gather kernel -> this one, us: 267 images 17x24, 158 -> 32, 5x5 1553 -> 93 (296 TFLOP/s);
// 148 images 56x12, 65 -> 32, 5x5 963 -> 81; 604 images 13x16, 96 -> 10, 3x3 578 -> 48; 149 images 14x43, 32 -> 32, 3x3
// (rows too wide for the LDS kernels) 94 -> 29; 3 images 7x13, 160 -> 14 31 -> 18; whole blocks, 256 images: 13x13 256 -> 256
// 103 (494 TFLOP/s), 27x27 64 -> 192 5x5 187 (613), both slower than with operands streamed into LDS (dfilter16b.hpp).
#pragma once
#include "owt_host.hpp"
#include "xfilter.hpp"

namespace owt {

// Eight images' raw values of B blocks of 32 rows (or columns), and the fragments made of them.
template <int B, bool PAIR> struct ImageRaw {
    static_assert(!PAIR || B == 2, "a pair is two blocks");
    static constexpr int NV = PAIR ? 8 : 8 * B;
    uint32_t v[NV];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, unsigned lane_off, unsigned off, unsigned image)
    {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            if constexpr (PAIR) v[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)lane_off, (int)(off + (unsigned)j * image), 0);
            else
#pragma unroll
                for (int b = 0; b < B; b++)
                    v[8 * b + j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)lane_off + 64 * b, (int)(off + (unsigned)j * image), 0);
        }
    }
    __device__ __forceinline__ uint4 words(int b) const
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if constexpr (PAIR) w[i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], b ? 0x07060302u : 0x05040100u);
            else w[i] = __builtin_amdgcn_perm(v[8 * b + 2 * i + 1], v[8 * b + 2 * i], 0x05040100u);
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};

// A value of four wavefronts, `stride` floats apart in LDS, added in pairs.
__device__ __forceinline__ float owt_shared_tile_sum(const float *red, int at, int stride)
{
    return (red[at] + red[at + stride]) + (red[at + 2 * stride] + red[at + 3 * stride]);
}

// The bias gradient of a tile's filters: a lane's half of the images, its wavefronts' positions.
template <int KB, bool ZP>
__device__ __forceinline__ void owt_images_db(const GemmParams &p, const float (&db)[KB], bool part, int split, int k0, int wave, float *red)
{
    const int lane = threadIdx.x & 63, li = lane & 31;
    __syncthreads();                                // everyone has read the tile's sums
#pragma unroll
    for (int kb = 0; kb < KB; kb++) red[(wave * KB + kb) * 64 + lane] = db[kb] + __shfl_xor(db[kb], 32);
    __syncthreads();
    if (wave || lane >= 32) return;
#pragma unroll
    for (int kb = 0; kb < KB; kb++) {
        const int k = k0 + (ZP ? 2 * li + kb : 32 * kb + li);
        if (k >= p.g.K) continue;
        const float v = owt_shared_tile_sum(red, kb * 64 + lane, KB * 64);
        if (part) p.dbias_partial[(size_t)split * p.M + k] = v;
        else p.dbias[k] = p.alpha * v + (p.beta != 0.f ? p.beta * p.dbias[k] : 0.f);
    }
}

// KB filter blocks x CB channel blocks x the S taps of one filter row per wavefront; ZP / XP: filters / channels in pairs.
template <int KB, int CB, int S, bool ZP, bool XP, bool MASKED>
__global__ void __launch_bounds__(256, ifilter16_occ(KB, CB, S)) ifilter16_kernel(const GemmParams p)
{
    constexpr int RING = S + 1;
    // raw columns in flight: all that the registers beside the accumulators hold
    constexpr int RAW = ImageRaw<CB, XP>::NV + ImageRaw<KB, ZP>::NV * (MASKED ? 2 : 1), SINGLE = (KB == 2 && !ZP) || (CB == 2 && !XP);
    constexpr int AHEAD = 16 * KB * CB * S + RAW * RING + (SINGLE ? 72 : 60) > 512 / ifilter16_occ(KB, CB, S) ? RING / 2 : RING;

    const Geom &g = p.g;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, split;
    if (!owt_split_major_wg(p.tiles_m * p.tiles_n, p.splits, tile, split)) return;
    const int kt = tile / p.tiles_n, rem = tile - kt * p.tiles_n;
    const int r = rem / p.ctiles, ct = rem - r * p.ctiles;
    const int k0 = kt * 32 * KB, c0 = ct * 32 * CB;

    // output rows whose input row p + r - pad_h exists, and this wavefront's range of (image group, row, column)
    const int p_lo = max(0, g.ph - r), Pv = max(0, min(g.P, g.H + g.ph - r) - p_lo), Q = g.Q;
    const int groups = (g.N + 15) >> 4, total = groups * Pv * Q;
    const int per = (total + p.splits - 1) / p.splits;
    const int g_beg = min(total, split * per), g_end = min(total, g_beg + per), sub = (per + 3) >> 2;
    const int o_beg = min(g_end, g_beg + wave * sub), o_end = min(g_end, o_beg + sub);

    // Byte offsets.  Images past the last are past the descriptor and read as zeros (the host has checked that no offset of a
    // group of 16 wraps round); channels and filters past a ragged tile read whatever is there and only reach accumulator
    // rows and columns that are never stored.
    const unsigned imgx = (unsigned)(g.H * g.W * g.C) * 2u, imgz = (unsigned)(g.P * Q * g.K) * 2u;
    const unsigned xall = imgx * (unsigned)g.N, zall = imgz * (unsigned)g.N;
    const unsigned xlane = (unsigned)(8 * lh) * imgx + (unsigned)(c0 + li * (XP ? 2 : 1)) * 2u;
    const unsigned zlane = (unsigned)(8 * lh) * imgz + (unsigned)(k0 + li * (ZP ? 2 : 1)) * 2u;
    const unsigned xstep = (unsigned)g.C * 2u, zstep = (unsigned)g.K * 2u;

    split_acc acc[KB][CB][S];
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int s = 0; s < S; s++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[kb][cb][s][e] = 0.f;
    float db[KB], row_db[KB];                       // the bias gradient; rows are summed by themselves, one long chain rounds more
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] = row_db[kb] = 0.f;
    const bool do_db = ct == 0 && r == g.ph && p.dbias != nullptr;        // every output row has an input row there

    // a row of the walk is len + S - 1 columns of x for len outputs; two places in the walk: where loads are issued and where
    // products are taken
    struct Place { int left, n0, prow, qa, i, len; };
    Place ld;
    {
        const int grp = o_beg / (Pv > 0 ? Pv * Q : 1), o = o_beg - grp * (Pv * Q);
        ld.left = o_end - o_beg; ld.n0 = 16 * grp; ld.prow = o / Q; ld.qa = o - ld.prow * Q; ld.i = 0;
        ld.len = min(Q - ld.qa, ld.left);
        ld.left -= ld.len;
    }
    Place at = ld;
    auto advance = [&](Place &w) __attribute__((always_inline)) {
        if (++w.i == w.len + S - 1) {
            w.i = 0;
            w.qa = 0;
            if (++w.prow == Pv) { w.prow = 0; w.n0 += 16; }
            w.len = min(Q, w.left);                 // 0 past the end of the walk: such rows load nothing and hold no products
            w.left -= w.len;
        }
    };
    const int rows = o_end > o_beg ? (o_end - 1) / Q - o_beg / Q + 1 : 0;
    const int steps = o_end - o_beg + rows * (S - 1);

    ImageRaw<CB, XP> xr[AHEAD];
    ImageRaw<KB, ZP> zr[AHEAD], yr[MASKED ? AHEAD : 1];
    auto load = [&](int i) __attribute__((always_inline)) {
        const int u = i % AHEAD;
        const int w = ld.qa - g.pw + ld.i, q = ld.i - (S - 1);
        const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(p.b, ld.len > 0 && (unsigned)w < (unsigned)g.W ? xall : 0u);
        xr[u].load(xrs, xlane, (unsigned)ld.n0 * imgx + (unsigned)((ld.prow + p_lo + r - g.ph) * g.W + w) * xstep, imgx);
        const unsigned zbytes = ld.len > 0 && q >= 0 ? zall : 0u;
        const unsigned zoff = (unsigned)ld.n0 * imgz + (unsigned)((ld.prow + p_lo) * Q + ld.qa + q) * zstep;
        zr[u].load(owt_make_rsrc(p.a, zbytes), zlane, zoff, imgz);
        if (MASKED) yr[MASKED ? u : 0].load(owt_make_rsrc(p.mask, zbytes), zlane, zoff, imgz);
        advance(ld);
    };
    uint4 win[RING][CB], az[2][KB];
    auto pack = [&](int u, int a) __attribute__((always_inline)) {
        const int i = u % AHEAD;
#pragma unroll
        for (int cb = 0; cb < CB; cb++) win[u][cb] = xr[i].words(cb);
#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            az[a][kb] = zr[i].words(kb);
            if (MASKED) az[a][kb] = mask_words16(az[a][kb], yr[MASKED ? i : 0].words(kb));
        }
        if (do_db) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++) row_db[kb] += sum8_bf16(az[a][kb]);
        }
    };

#pragma unroll
    for (int u = 0; u < AHEAD; u++) load(u);
    pack(0, 0);
    load(0);
    static_assert(RING % 2 == 0, "the two sets of dz fragments alternate");
    for (int t = 0; t < steps; t += RING) {
#pragma unroll
        for (int u = 0; u < RING; u++) {
            // the column of step t + u has been packed; behind its products the next one's is packed and its raw registers are
            // loaded again
            const bool has = at.i >= S - 1 && at.len > 0, row_end = at.i == at.len + S - 2;
            advance(at);
            const int nx = (u + 1) % RING;
            if (has) {
#pragma unroll
                for (int s = 0; s < S; s++)
#pragma unroll
                    for (int kb = 0; kb < KB; kb++)
#pragma unroll
                        for (int cb = 0; cb < CB; cb++)
                            acc[kb][cb][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(split_frag, az[u & 1][kb]), __builtin_bit_cast(split_frag, win[(u + 2 + s) % RING][cb]), acc[kb][cb][s], 0, 0, 0);
                if (do_db && row_end) {
#pragma unroll
                    for (int kb = 0; kb < KB; kb++) { db[kb] += row_db[kb]; row_db[kb] = 0.f; }
                }
            }
            pack(nx, (u + 1) & 1);
            load(nx);
        }
    }
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] += row_db[kb];

    // register e of lane (li, lh): row 8*(e/4) + 4*lh + e%4 of its filter block, column li of its channel block
    const bool part = p.splits > 1;
    float *out = part ? p.partial + (size_t)split * p.M * p.Ncols : (float *)p.out;
    const int RS = g.R * S;
    auto store = [&](int kb, int s, int e, int c, float v) __attribute__((always_inline)) {
        const int row = 8 * (e / 4) + 4 * lh + e % 4, k = k0 + (ZP ? 2 * row + kb : 32 * kb + row);
        if (k >= g.K) return;
        const size_t o = ((size_t)k * RS + r * S + s) * g.C + c;
        if (part) out[o] = v;
        else out[o] = p.alpha * v + (p.beta != 0.f ? p.beta * out[o] : 0.f);
    };
    __shared__ float red[4 * S * 16 * 64];
#pragma unroll
    for (int cb = 0; cb < CB; cb++) {
        const int c = c0 + (XP ? 2 * li + cb : 32 * cb + li);
#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            if (cb + kb) __syncthreads();           // everyone has read the block before
#pragma unroll
            for (int s = 0; s < S; s++)
#pragma unroll
                for (int e = 0; e < 16; e++) red[((wave * S + s) * 16 + e) * 64 + lane] = acc[kb][cb][s][e];
            __syncthreads();
            for (int v = wave; v < S * 16; v += 4) {
                const float sum = owt_shared_tile_sum(red, v * 64 + lane, S * 16 * 64);
                if (c < g.C) store(kb, v / 16, v % 16, c, sum);
            }
        }
    }
    if (do_db) owt_images_db<KB, ZP>(p, db, part, split, k0, wave, red);
}

}  // namespace owt
