// Stride-1 filter gradient, bf16 storage, channels and filters in eights: reduction over images, operands streamed into LDS.
//
//   dw[k][r][s][c] = sum over (p,q) of  sum over images n of  dz[n,p,q,k] * x[n, p+r-pad_h, q+s-pad_w, c]
//
// (Section 4 of the paper, backward step 2.)  As in ifilter16.hpp a 16-deep matrix instruction takes 16 images at one output
// position, so a filter tap is the neighbouring position's fragment: walking along a row, a wavefront reads the fragments of ONE
// column of x and of dz from LDS per position and has those of the last S columns in registers.  The kernels with the reduction over
// pixels (dfilter16b.hpp) read every tap's fragment anew: 1.7 transposing 8-byte reads a matrix instruction for 3 taps and 2.4 for 5,
// where LDS delivers about 1.7; here 0.7 to 1 and 0.6 to 0.8.
//  * An instruction loads 16 images x 32 channels of one position, 1 KB, straight into LDS, where a transposing read's four rows
//    are 256 contiguous bytes (no bank conflict; the counters show none).  The loads of a stage (L positions) are issued NST - 1
//    stages ahead; one barrier a stage.  Half of a SIMD's wavefronts take it in front of the products of a stage's last position and
//    half behind them, so that these cover the others' wait: 5x5, 1024 images, 384 -> 368 us, 3x3 384 -> 256 258 -> 254.
//  * The walk needs next to no scalar instructions (with positions counted one by one, 75 a position, 5x5 took 520 us and not
//    390): rows are rounded up to whole stages, what a row starts with is worked out once a row, lanes keep their part of a load's
//    offset, and there is one branch around a position's products, for the S - 1 columns left of the first.  (Products of taps
//    outside the image left out one by one: the accumulators are copied at every branch, 1600 registers spilled.)
//  * Filter rows outside the image are not walked over.
//
// What bounds it: at 1024 images the matrix unit is busy 50 to 58 % of the time at 2.0 to 2.15 GHz, whichever tile, ring or number of
// work-groups to a CU (16 forms within 6 % of each other); without the loads 5 to 20 % faster.  Partial sums take 20 to 30 us of 100
// MB at one tile a CU.  Measured with the reduce pass, us, dfilter16b -> here: 13x13, 1024 images, 384 -> 256 331 -> 256 (1196 TFLOP/s),
// 192 -> 384 214 -> 201; 27x27, 64 -> 192 5x5, 256 images 153 -> 108, 1024 images 444 -> 375 (1225).  210 drawn layers of channels in
// eights, with the choice of kernel: 7900 -> 6398; error of dw against 64 bits 0.93 times the kernels before on average (43 layers,
// at most 1.11).
#pragma once
#include <type_traits>

#include "dfilter_bf16.hpp"
#include "owt_host.hpp"
#include "split3.hpp"

namespace owt {

// KB filter blocks x CB channel blocks x the S taps of one filter row per wavefront, WK x WC wavefronts; a stage of the LDS ring
// is L steps, NST stages, OCC work-groups per CU.
template <int KB, int CB, int S, int WK, int WC, int L, int NST, int OCC>
__global__ void __launch_bounds__(64 * WK * WC, OCC * WK * WC / 4) ifilter16b_kernel(const GemmParams p)
{
    constexpr int NW = WK * WC, KBLK = KB * WK, CBLK = CB * WC, BLK = KBLK + CBLK, KT = 32 * KBLK, CT = 32 * CBLK;
    constexpr int RING = S + 1, PIECES = L * BLK, STAGEB = PIECES * 1024;
    constexpr int ZL = (L * KBLK + NW - 1) / NW, SLOTS = ZL + (L * CBLK + NW - 1) / NW;    // a wavefront's loads of dz in a stage, at most, and of both
    constexpr int LPW = (PIECES + NW - 1) / NW;                                             // and what it issues in all, or one less
    static_assert(RING % L == 0 && RING % 2 == 0, "the unrolled walk holds whole stages");
    static_assert(NST >= 3, "one stage is read, one has landed, one is in flight");
    static_assert((NST - 2) * LPW < 64, "the vector-memory counter holds the loads in flight");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGEB];

    const Geom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int wkw = wave / WC, wcw = wave % WC;
    int tile, split;
    if (!owt_split_major_wg(p.tiles_m * p.tiles_n, p.splits, tile, split)) return;
    const int kt = tile / p.tiles_n, rem = tile - kt * p.tiles_n;
    const int r = rem / p.ctiles, ct = rem - r * p.ctiles;
    const int k0 = kt * KT, c0 = ct * CT;

    // output rows whose input row p + r - pad_h exists, and this work-group's range of (image group, row, column)
    const int p_lo = max(0, g.ph - r), Pv = max(0, min(g.P, g.H + g.ph - r) - p_lo), Q = g.Q;
    const int total = ((g.N + 15) >> 4) * Pv * Q;
    const int per = (total + p.splits - 1) / p.splits;
    const int o_beg = min(total, split * per), o_end = min(total, o_beg + per);

    const unsigned imgx = (unsigned)(g.H * g.W * g.C) * 2u, imgz = (unsigned)(g.P * Q * g.K) * 2u;
    const unsigned xall = imgx * (unsigned)g.N, zall = imgz * (unsigned)g.N;
    const unsigned xstep = (unsigned)g.C * 2u, zstep = (unsigned)g.K * 2u;

    // A row of the walk [qa, qa + len) takes the columns w of x from qa - pad_w, where its first output's first tap is, to its last
    // output's last tap: len + S - 1 steps, and as many more as make whole stages; output w - (S - 1) + pad_w goes with column w.
    // (Before the first output and after the last there are no products: what dz holds there does not matter.)
    struct Row { int left, n0, prow, qa, len; };
    auto start_row = [&](Row &a) __attribute__((always_inline)) {
        a.len = min(Q - a.qa, a.left);              // 0 past the end of the walk
        a.left -= a.len;
    };
    auto next_row = [&](Row &a) __attribute__((always_inline)) {
        a.qa = 0;
        if (++a.prow == Pv) { a.prow = 0; a.n0 += 16; }
        start_row(a);
    };
    Row at;
    {
        const int grp = o_beg / max(1, Pv * Q), o = o_beg - grp * (Pv * Q);
        at.left = __builtin_amdgcn_readfirstlane(o_end - o_beg);      // (wave-uniform: the walk stays in scalar registers)
        at.n0 = __builtin_amdgcn_readfirstlane(16 * grp);
        at.prow = __builtin_amdgcn_readfirstlane(o / Q);
        at.qa = __builtin_amdgcn_readfirstlane(o - at.prow * Q);
        start_row(at);
    }

    // Loads: an instruction takes 16 images x 32 channels of one position, lane l image l / 4, channels 8 (l % 4) ..; a stage is
    // [step][dz blocks] [step][x blocks], its instructions dealt to the wavefronts round robin.
    unsigned voff[SLOTS], fill_at = 0;
    int lstep[SLOTS];
    const int xwave = (wave + NW - L * KBLK % NW) % NW;
#pragma unroll
    for (int i = 0; i < SLOTS; i++) {
        const bool isx = i >= ZL;
        const int j = isx ? xwave + NW * (i - ZL) : wave + NW * i, blk = j % (isx ? CBLK : KBLK);
        lstep[i] = j / (isx ? CBLK : KBLK);
        voff[i] = (unsigned)(lane >> 2) * (isx ? imgx : imgz) + (unsigned)((isx ? c0 : k0) + blk * 32 + (lane & 3) * 8) * 2u + (unsigned)lstep[i] * (isx ? xstep : zstep);
    }
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const owt_i32x4 xrs = make_rsrc(p.b, xall), zrs = make_rsrc(p.a, zall);
    // what a stage's loads need: byte offsets of its first column in x and in dz, that column, the column the row ends at
    Row ld = at;
    int lw, lend;
    unsigned xo, zo;
    auto load_row = [&]() __attribute__((always_inline)) {
        lw = ld.qa - g.pw;
        lend = ld.len > 0 ? lw + ld.len + S - 1 : 0x40000000;      // past the end of the walk: nothing of x
        if (ld.len == 0) lw = 0x20000000;
        xo = (unsigned)ld.n0 * imgx + (unsigned)((ld.prow + p_lo + r - g.ph) * g.W + lw) * xstep;
        zo = (unsigned)ld.n0 * imgz + (unsigned)((ld.prow + p_lo) * Q + lw - (S - 1) + g.pw) * zstep;
    };
    load_row();
    auto issue = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < SLOTS; i++) {
            const bool isx = i >= ZL;
            const int n = isx ? i - ZL : i, have = L * (isx ? CBLK : KBLK), j = (isx ? xwave : wave) + NW * n;
            if ((n + 1) * NW > have && j >= have) continue;
            owt_i32x4 rs = isx ? xrs : zrs;
            if (isx) rs.z = __builtin_amdgcn_readfirstlane((unsigned)(lw + lstep[i]) < (unsigned)g.W ? (int)xall : 0);
            // (the sum in 32 bits: a stage may begin left of the row, and of the tensor)
            buffer_load16_to_lds(rs, voff[i] + (isx ? xo : zo), lds_base + fill_at + (unsigned)(isx ? L * KBLK + j : j) * 1024u);
        }
        fill_at += STAGEB;
        if (fill_at >= NST * STAGEB) fill_at -= NST * STAGEB;
        lw += L;
        xo += L * xstep;
        zo += L * zstep;
        if (lw >= lend) { next_row(ld); load_row(); }
    };
    // Waits until at most N of this wavefront's stages are still on their way and all it has read from LDS is in registers, and for the
    // others'.  What is loaded next goes into the stage before the one that is left here.  Its last fragments may not have been used: where a
    // row begins or ends there are whole stages without products, which are what else would have waited for them.
    const bool fewer = wave >= PIECES % NW;
    auto arrived = [&](auto n) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value, A = N * LPW, B = N * (LPW - 1);
        asm volatile("" ::: "memory");
        if (PIECES % NW && fewer) __builtin_amdgcn_s_waitcnt((B & 15) | ((B >> 4) << 14) | 0x0070);      // lgkmcnt(0), expcnt untouched
        else __builtin_amdgcn_s_waitcnt((A & 15) | ((A >> 4) << 14) | 0x0070);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    float16v acc[KB][CB][S];
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
    int turn = wcw;                                 // the wavefronts that hold the same filters take turns in summing them

    // transposing reads: a lane's source position of a 16 x 32 block (image, channel), the second read four images further on
    const int grp16 = lane >> 4, i16 = lane & 15;
    const unsigned tr_lane = (unsigned)((8 * (grp16 >> 1) + (i16 >> 2)) * 64 + 32 * (grp16 & 1) + 8 * (i16 & 3));
    unsigned zrd = lds_base + tr_lane + (unsigned)(KB * wkw) * 1024u, xrd = lds_base + tr_lane + (unsigned)(L * KBLK + CB * wcw) * 1024u;
    typedef __attribute__((address_space(3))) short4_t *lds_frag_ptr;
    auto frag = [](unsigned at) __attribute__((always_inline)) {
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_frag_ptr)(size_t)at);
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_frag_ptr)(size_t)(at + 256u));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    const bool late = (wave >> 2) & 1;
    unsigned rd = 0;                                // the stage that fragments are read from
    short8_t win[RING][CB], az[2][KB];

#pragma unroll
    for (int i = 0; i < NST - 1; i++) issue();
    arrived(std::integral_constant<int, NST - 2>{});
#pragma unroll
    for (int cb = 0; cb < CB; cb++) win[0][cb] = frag(xrd + cb * 1024);
#pragma unroll
    for (int kb = 0; kb < KB; kb++) az[0][kb] = frag(zrd + kb * 1024);

    int i0 = -(S - 1);                              // this stage's first step, counted from the row's first output
    while (at.len > 0) {
#pragma unroll
        for (int u = 0; u < RING; u++) {
            // The fragments of step t + u are in registers; those of the next one are read behind its products.  At the last step of a
            // stage the next stage has to land and the one before is free: half of a SIMD's wavefronts wait and issue loads in front
            // of the step's products, the others behind them, so that the matrix unit is not left by all of them at a time.
            const int nx = (u + 1) % RING, nst = (u + 1) % L;
            const bool last = u % L == L - 1;
            auto read_next = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int cb = 0; cb < CB; cb++) win[nx][cb] = frag(rd + xrd + (unsigned)(nst * CBLK + cb) * 1024u);
#pragma unroll
                for (int kb = 0; kb < KB; kb++) az[(u + 1) & 1][kb] = frag(rd + zrd + (unsigned)(nst * KBLK + kb) * 1024u);
            };
            const bool has = (unsigned)(i0 + u % L) < (unsigned)at.len;
            if (last && !late) {
                arrived(std::integral_constant<int, NST - 3>{});
                issue();
            }
            if (!last) read_next();
            if (has) {
#pragma unroll
                for (int s = 0; s < S; s++)
#pragma unroll
                    for (int kb = 0; kb < KB; kb++)
#pragma unroll
                        for (int cb = 0; cb < CB; cb++)
                            acc[kb][cb][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, az[u & 1][kb]),
                                                                                    __builtin_bit_cast(bf16x8_t, win[(u + 2 + s) % RING][cb]), acc[kb][cb][s], 0, 0, 0);
            }
            if (last) {
                if (late) {
                    arrived(std::integral_constant<int, NST - 3>{});
                    issue();
                }
                rd += STAGEB;
                if (rd >= NST * STAGEB) rd -= NST * STAGEB;
                read_next();
            }
            if (do_db) {
                if (has && turn == 0) {
#pragma unroll
                    for (int kb = 0; kb < KB; kb++) row_db[kb] += sum8_bf16(__builtin_bit_cast(uint4, az[u & 1][kb]));
                }
                turn = turn == 0 ? WC - 1 : turn - 1;
            }
            if (u % L == L - 1) {
                i0 += L;
                if (i0 >= at.len) {
                    i0 = -(S - 1);
                    next_row(at);
#pragma unroll
                    for (int kb = 0; kb < KB; kb++) { db[kb] += row_db[kb]; row_db[kb] = 0.f; }
                }
            }
        }
    }

    // register e of lane (li, lh): filter 8*(e/4) + 4*lh + e%4 of its block, channel li.  Filters past the last are past the
    // descriptor, channels past the last get an offset outside it.
    const bool part = p.splits > 1;
    const __amdgpu_buffer_rsrc_t ors = owt_make_rsrc(part ? p.partial + (size_t)split * p.M * p.Ncols : (float *)p.out, (unsigned)p.M * (unsigned)p.Ncols * 4u);
    const unsigned kstep = (unsigned)p.Ncols * 4u;
    auto store = [&](auto form) __attribute__((always_inline)) {       // 0: partial sums, 1: scaled, 2: scaled and added to what is there
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            const int c = c0 + (CB * wcw + cb) * 32 + li;
            const unsigned at_c = c < g.C ? (unsigned)(k0 + KB * wkw * 32 + 4 * lh) * kstep + (unsigned)(r * S * g.C + c) * 4u : 0x80000000u;
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int e = 0; e < 16; e++)
#pragma unroll
                    for (int s = 0; s < S; s++) {
                        const unsigned so = (unsigned)(kb * 32 + 8 * (e / 4) + e % 4) * kstep + (unsigned)s * 2u * xstep;
                        float v = acc[kb][cb][s][e];
                        if (decltype(form)::value > 0) v *= p.alpha;
                        if (decltype(form)::value > 1) v += p.beta * __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ors, (int)at_c, (int)so, 0));
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ors, (int)at_c, (int)so, 0);
                    }
        }
    };
    if (part) store(std::integral_constant<int, 0>{});
    else if (p.beta == 0.f) store(std::integral_constant<int, 1>{});
    else store(std::integral_constant<int, 2>{});
    __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): the last loads into LDS have landed, too
    if (do_db) {                                    // uniform over the work-group
        __syncthreads();
        float *red = (float *)lds;                  // [wavefront column][filter]
#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            const float both = db[kb] + __shfl_xor(db[kb], 32);
            if (lh == 0) red[wcw * KT + (KB * wkw + kb) * 32 + li] = both;
        }
        __syncthreads();
        for (int i = tid; i < KT; i += 64 * NW) {
            const int k = k0 + i;
            if (k >= g.K) continue;
            float v = 0.f;
#pragma unroll
            for (int j = 0; j < WC; j++) v += red[j * KT + i];
            if (part) p.dbias_partial[(size_t)split * p.M + k] = v;
            else p.dbias[k] = p.alpha * v + (p.beta != 0.f ? p.beta * p.dbias[k] : 0.f);
        }
    }
}

}  // namespace owt
