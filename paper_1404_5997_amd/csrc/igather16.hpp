// Filter gradient of any convolution, bf16 storage, with the reduction over images.
//
//   dw[k][j] = sum over (p,q), images n of  dz[n,p,q,k] * x[n, p*sh + r - pad_h, q*sw + s - pad_w, c],   j = (r*S + s)*C + c
//
// (Section 4 of the paper, backward step 2.)  ifilter16.hpp's operands (16 images at one position, as they are loaded) with
// xgather.hpp's columns: the filter's (r, s, c) places packed densely, a lane keeping its place's offset and (r, s), so any
// stride and any channel count will do.  Neighbouring positions share nothing here, so a wavefront's KB x CB blocks cost
// 8 * CB loads of 2 bytes and 8 * KB of dz (8 of 4 bytes for two blocks of an even number of filters) per position, and those
// bound it.  Raw loads run four positions ahead, two where registers are short (with four, the
// 64-filter tile spilled 56 registers and took 285 us where it takes 136).
// Takes what the strided kernels that stage rows in LDS (sfilter_bf16.hpp, sfilter16b.hpp) do not: rows that are no multiple of
// four values, odd filter counts, other strides and taps.
// Work-groups of four wavefronts a tile as in ifilter16.hpp; 91 layers 2113 -> 1744 us.  With them two blocks of places beside
// three, which leave less of a tile idle.
// Measured with the reduce pass, a tile to a wavefront, gather kernel on the fp32 instruction -> this one, us: first layers, 332 images 179x179x3 -> 48, 11x11
// stride 4 1466 -> 136 (164 TFLOP/s), 72 images 133x133x3 -> 96, 7x7 208 -> 36, 54 images 83x83x3 -> 64 62 -> 27, 3 images 75x75x3 30 -> 13;
// 1x1, 187 images 44x55, 21 -> 96 333 -> 58.
#pragma once
#include "ifilter16.hpp"

namespace owt {

template <int KB, int CB, bool ZP, bool MASKED>
__global__ void __launch_bounds__(256, KB == 2 && !ZP && MASKED ? 1 : 2) igather16_kernel(const GemmParams p)
{
    constexpr int AHEAD = MASKED || KB == 2 ? 2 : 4;

    const Geom &g = p.g;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile, split;
    if (!owt_split_major_wg(p.tiles_m * p.tiles_n, p.splits, tile, split)) return;
    const int kt = tile / p.tiles_n, ct = tile - kt * p.tiles_n;
    const int k0 = kt * 32 * KB, j0 = ct * 32 * CB;

    const int P = g.P, Q = g.Q, total = ((g.N + 15) >> 4) * P * Q;
    const int per = p.ksteps_per_split, g_beg = min(total, split * per), g_end = min(total, g_beg + per), sub = (per + 3) >> 2;
    const int o_beg = min(g_end, g_beg + wave * sub), o_end = min(g_end, o_beg + sub);

    // what must read as zero gets an offset of xall, the end of the tensor; with the scalar part added it stays below 2^32
    // (host-checked), as do the offsets of images past the last.  Ragged tiles: as in ifilter16.hpp.
    const unsigned imgx = (unsigned)(g.H * g.W * g.C) * 2u, imgz = (unsigned)(P * Q * g.K) * 2u;
    const unsigned xall = imgx * (unsigned)g.N, zall = imgz * (unsigned)g.N;
    const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(p.b, xall);
    int coff[CB], cr[CB], cs[CB];
#pragma unroll
    for (int cb = 0; cb < CB; cb++) {
        const int j = j0 + cb * 32 + li, rs = g.dC.div(j), r = g.dS.div(rs);
        cr[cb] = j < p.Ncols ? r : 0x10000000;
        cs[cb] = rs - r * g.S;
        coff[cb] = ((r * g.W + cs[cb]) * g.C + (j - rs * g.C)) * 2 + (int)((unsigned)(8 * lh) * imgx);
    }
    const unsigned zlane = (unsigned)(8 * lh) * imgz + (unsigned)(k0 + li * (ZP ? 2 : 1)) * 2u;

    split_acc acc[KB][CB];
#pragma unroll
    for (int kb = 0; kb < KB; kb++)
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[kb][cb][e] = 0.f;
    float db[KB], run_db[KB];                       // the bias gradient; runs of 16 positions are summed by themselves
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] = run_db[kb] = 0.f;
    const bool do_db = ct == 0 && p.dbias != nullptr;

    int o = o_beg, n0, pp, qq;                      // the position that loads are issued for
    {
        const int grp = o_beg / (P * Q), rem = o_beg - grp * (P * Q);
        n0 = 16 * grp; pp = rem / Q; qq = rem - pp * Q;
    }
    uint32_t xr[AHEAD][CB][8];
    ImageRaw<KB, ZP> zr[AHEAD], yr[MASKED ? AHEAD : 1];
    auto load = [&](int u) __attribute__((always_inline)) {
        const int h0 = pp * g.sh - g.ph, w0 = qq * g.sw - g.pw;
        const bool live = o < o_end;
        // the corner may lie outside the image: its offset is folded into the lanes' part, modulo 2^32
        const unsigned xoff = live ? (unsigned)n0 * imgx : 0u;
        const int corner = (h0 * g.W + w0) * g.C * 2;
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            const bool in = (unsigned)(h0 + cr[cb]) < (unsigned)g.H && (unsigned)(w0 + cs[cb]) < (unsigned)g.W;
            const unsigned place = live && in ? (unsigned)(coff[cb] + corner) : xall;
#pragma unroll
            for (int e = 0; e < 8; e++)
                xr[u][cb][e] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xrs, (int)place, (int)(xoff + (unsigned)e * imgx), 0);
        }
        const unsigned zoff = (unsigned)n0 * imgz + (unsigned)((pp * Q + qq) * g.K) * 2u, zbytes = live ? zall : 0u;
        zr[u].load(owt_make_rsrc(p.a, zbytes), zlane, zoff, imgz);
        if (MASKED) yr[MASKED ? u : 0].load(owt_make_rsrc(p.mask, zbytes), zlane, zoff, imgz);
        o++;
        const bool row_end = qq + 1 == Q, image_end = row_end && pp + 1 == P;
        qq = row_end ? 0 : qq + 1;
        pp = image_end ? 0 : (row_end ? pp + 1 : pp);
        n0 = image_end ? n0 + 16 : n0;
    };
    uint4 bx[CB], az[KB];
    auto pack = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            const uint32_t (&v)[8] = xr[u][cb];
            bx[cb] = make_uint4(__builtin_amdgcn_perm(v[1], v[0], 0x05040100u), __builtin_amdgcn_perm(v[3], v[2], 0x05040100u),
                                __builtin_amdgcn_perm(v[5], v[4], 0x05040100u), __builtin_amdgcn_perm(v[7], v[6], 0x05040100u));
        }
#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            az[kb] = zr[u].words(kb);
            if (MASKED) az[kb] = mask_words16(az[kb], yr[MASKED ? u : 0].words(kb));
        }
        if (do_db) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++) run_db[kb] += sum8_bf16(az[kb]);
        }
    };
#pragma unroll
    for (int u = 0; u < AHEAD; u++) load(u);
    // (past the walk's end a position's operands are zeros)
    for (int i = o_beg; i < o_end; i += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            pack(u);
            load(u);
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int cb = 0; cb < CB; cb++)
                    acc[kb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(split_frag, az[kb]), __builtin_bit_cast(split_frag, bx[cb]),
                                                                          acc[kb][cb], 0, 0, 0);
        }
        if (do_db && ((i - o_beg) & 15) >= 16 - AHEAD) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++) { db[kb] += run_db[kb]; run_db[kb] = 0.f; }
        }
    }
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] += run_db[kb];

    // register e of lane (li, lh): row 8*(e/4) + 4*lh + e%4 of its filter block, place li of its block
    const bool part = p.splits > 1;
    float *out = part ? p.partial + (size_t)split * p.M * p.Ncols : (float *)p.out;
    auto store = [&](int kb, int cb, int e, float v) __attribute__((always_inline)) {
        const int row = 8 * (e / 4) + 4 * lh + e % 4, k = k0 + (ZP ? 2 * row + kb : 32 * kb + row), j = j0 + cb * 32 + li;
        if (k >= g.K || j >= p.Ncols) return;
        const size_t at = (size_t)k * p.Ncols + j;
        if (part) out[at] = v;
        else out[at] = p.alpha * v + (p.beta != 0.f ? p.beta * out[at] : 0.f);
    };
    __shared__ float red[4 * CB * 16 * 64];
#pragma unroll
    for (int kb = 0; kb < KB; kb++) {
        if (kb) __syncthreads();
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int e = 0; e < 16; e++) red[((wave * CB + cb) * 16 + e) * 64 + lane] = acc[kb][cb][e];
        __syncthreads();
        for (int v = wave; v < CB * 16; v += 4) store(kb, v / 16, v % 16, owt_shared_tile_sum(red, v * 64 + lane, CB * 16 * 64));
    }
    if (do_db) owt_images_db<KB, ZP>(p, db, part, split, k0, wave, red);
}

}  // namespace owt
