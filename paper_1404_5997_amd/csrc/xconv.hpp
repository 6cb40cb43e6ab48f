// Direct stride-1 convolution, fp32 storage, on the bf16 matrix unit with operands split in three (split3.hpp):
// forward and backward-data of the stride-1 layers (Section 4 of the paper, forward step 2 / backward step 2).
//
// Panel-resident like dconv.hpp: the input pixels under a tile of BM consecutive output pixels are one contiguous run
// of NHWC pixels, loaded once per 16-channel chunk and read by every filter tap at a shifted row.  What bounds it is
// the matrix pipe (six 32-cycle instructions per 32x32x16 block product), so everything else is arranged around that:
//  * a wavefront owns 64 pixels x 64 filters: 2 x 2 blocks with two accumulators each (128 registers), and per tap and
//    chunk it reads 6 + 6 fragments of 1 KB for 24 matrix instructions (half a fragment per instruction; the LDS could
//    deliver about one), two wavefronts per SIMD;
//  * the panel's values are split once, on their way from global memory into LDS (R*S taps and the tile's filter blocks
//    reuse them): 7 vector instructions per value, 4-8 % of the matrix time for a 3x3 layer, where writing the three
//    parts to memory and reading them back would move 10 bytes per value;
//  * the filters are split and laid out once per call in the order the fragments are read (xconv_pack_kernel), so a
//    tap's slice is a few 1 KB pieces that go straight into LDS, and a fragment read is 64 consecutive 16-byte pieces;
//  * the panel is kept as six planes (part, 8-channel half) of one 16-byte piece per pixel: a fragment read of 32
//    consecutive pixels is 512 consecutive bytes whatever the tap's shift.  The counters still show bank conflicts in 19-25 %
//    of the LDS cycles: planes are PR + 1 = 1 (mod 8) pieces apart, so the two halves of a pixel, which neighbouring threads
//    store, meet in one bank group;
//  * slices sit in a ring of four: one barrier per tap is enough, a slice has two taps' time to arrive, and the fragments
//    of a tap are read during the tap before, each into the registers of a fragment that has just had its last product.
// Taps that fall outside the image read the row of zeros behind each plane.
// Measured, 128 images, kernel on the fp32 instruction -> this one, us: forward 3x3 192->384 218 -> 127 (226 TFLOP/s), 256->256
// 218 -> 128, 384->256 320 -> 187, 5x5 64->192 453 -> 250; backward-data 232 -> 142, - , - , 444 -> 260.  With each tap's
// fragments read behind the tap's own barrier instead of during the tap before (and the panel twice): 135, 136, 198, 255.
//
// A strided forward pass of few channels (the first layer) runs here, too, seen over blocks of sh x sw input pixels: 11 x 11
// taps of 3 channels at stride 4 are 3 x 3 taps of 48 channels, 432 reduction steps for 363.  Measured, 128 images of
// 224x224x3 -> 64: 170 us on the fp32 instruction, 123 here (146 TFLOP/s on the 363); half of the time goes to the panel's
// 4-byte loads, the prologue and the stores of work-groups that have only 27 steps.
#pragma once
#include "igemm.hpp"
#include "split3.hpp"

namespace owt {

// Filters -> [chunk][tap][32-column block][part][lane][8 values], zero-padded: column = 32 * block + lane % 32 (a filter
// in forward, an input channel in backward-data), reduction index = 16 * chunk + 8 * (lane / 32) + j.  Backward-data
// reads w[k][R-1-r][S-1-s][c] with k as the reduction index.  One thread per (chunk, tap, block, lane).
template <bool BWD>
__global__ void __launch_bounds__(256) xconv_pack_kernel(const float *__restrict__ w, uint4 *__restrict__ out, int K, int RS,
                                                         int C, int chunks, int nblocks)
{
    const int total = chunks * RS * nblocks * 64;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        const int lane = i & 63, q = i >> 6, nb = q % nblocks, ct = q / nblocks, tap = ct % RS, ch = ct / RS;
        const int col = nb * 32 + (lane & 31), red = ch * 16 + (lane >> 5) * 8;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int kd = red + j;
            if (BWD) v[j] = (col < C && kd < K) ? w[((size_t)kd * RS + (RS - 1 - tap)) * C + col] : 0.f;
            else v[j] = (col < K && kd < C) ? w[((size_t)col * RS + tap) * C + kd] : 0.f;
        }
        uint4 h, m, l;
        split3_scaled(v, h, m, l);
        uint4 *o = out + (size_t)q * 192 + lane;
        o[0] = h; o[64] = m; o[128] = l;
    }
}

// The same for a strided forward pass seen as a stride-1 one over blocks of sh x sw pixels: the reduction index is
// (dy, dx, c) inside a block, the tap (rb, sb) names the block, and w[k][sh*rb + dy][sw*sb + dx][c] is zero past R or S.
static __global__ void __launch_bounds__(256) xconv_pack_blocks_kernel(const float *__restrict__ w, uint4 *__restrict__ out, Geom g, int RB,
                                                                int SB, int chunks, int nblocks)
{
    const int RS = RB * SB, total = chunks * RS * nblocks * 64, rowc = g.sw * g.C;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        const int lane = i & 63, q = i >> 6, nb = q % nblocks, ct = q / nblocks, tap = ct % RS, ch = ct / RS;
        const int col = nb * 32 + (lane & 31), red = ch * 16 + (lane >> 5) * 8, rb = tap / SB, sb = tap - rb * SB;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int kd = red + j, dy = kd / rowc, rem = kd - dy * rowc, dx = rem / g.C, c = rem - dx * g.C;
            const int r = rb * g.sh + dy, s = sb * g.sw + dx;
            v[j] = (col < g.K && dy < g.sh && r < g.R && s < g.S) ? w[((size_t)(col * g.R + r) * g.S + s) * g.C + c] : 0.f;
        }
        uint4 h, m, l;
        split3_scaled(v, h, m, l);
        uint4 *o = out + (size_t)q * 192 + lane;
        o[0] = h; o[64] = m; o[128] = l;
    }
}

// How a panel's values are loaded: XC_SCALAR 4 bytes at a time (any channel count), XC_VEC 16 bytes (channels a multiple of
// four), XC_BLOCKS a strided forward pass whose panel rows are blocks of sh x sw input pixels (p.g.R, p.g.S and the
// frame Hi, Wi, Ho, Wo, Cred count in blocks; p.g.H, W, C, strides and padding are the layer's own).
enum { XC_SCALAR = 0, XC_VEC = 1, XC_BLOCKS = 2 };

// WM x WN wavefronts of 32*MB pixels x 64 filters; PR panel rows; OCC wavefronts per SIMD the registers are cut for; MASKED: dy is masked by y > 0 on its way in.  At most
// 32 taps; 32-bit byte offsets in every tensor (host-checked).
template <class Epi, bool BWD, int WM, int WN, int MB, int PR, int OCC, int LOAD, bool MASKED>
__global__ void __launch_bounds__(64 * WM * WN, OCC) xconv_kernel(const GemmParams p)
{
    constexpr int NW = WM * WN, NT = 64 * NW, BM = 32 * MB * WM, BN = 64 * WN;
    constexpr int PL = PR + 1, PANEL = 6 * PL;                       // 16-byte units: a plane, a panel buffer
    constexpr int SL = BN / 32 * 3;                                  // 1 KB pieces of a filter slice
    constexpr int PU = (2 * PR + NT - 1) / NT;                       // (row, half) pairs of the panel per thread
    constexpr unsigned OOB = 0x80000000u;                            // a byte offset no descriptor here reaches

    __shared__ __attribute__((aligned(1024))) uint4 slices[4 * SL * 64];
    __shared__ __attribute__((aligned(16))) uint4 panel[PANEL];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int wm = wave / WN, wn = wave - wm * WN;

    const int ntiles = p.tiles_m * p.tiles_n;
    const int b = blockIdx.x, xcd = b & 7;
    const int logical = xcd * (ntiles >> 3) + min(xcd, ntiles & 7) + (b >> 3);
    const int tm = logical / p.tiles_n, tn = logical - tm * p.tiles_n;
    const int n0 = tn * BN;
    // pixel tiles run through the whole batch, or (p.tpi > 0) start anew with every image: a tile that straddles two images
    // of a pass without padding has the rows under the first one's last taps in its panel, too
    const int img = p.tpi > 0 ? tm / p.tpi : 0, hw = p.Ho * p.Wo;
    const int m0 = p.tpi > 0 ? img * hw + (tm - img * p.tpi) * BM : tm * BM, mlim = p.tpi > 0 ? (img + 1) * hw : p.M;
    const int split = blockIdx.y;
    const int ch_beg = split * p.ksteps_per_split, ch_end = min(p.ksteps, ch_beg + p.ksteps_per_split);

    const int R = p.g.R, S = p.g.S, RS = R * S, Hi = p.Hi, Wi = p.Wi, Cred = p.Cred;
    const int HoWo = p.Ho * p.Wo;

    auto pin = [&](int m, int &hh, int &ww) {
        const int n = p.dHoWo.div(m), rem = m - n * HoWo;
        const int ho = p.dWo.div(rem), wo = rem - ho * p.Wo;
        hh = ho - p.pah; ww = wo - p.paw;
        return n * Hi * Wi + hh * Wi + ww;
    };
    int th, tw;
    const int ps = pin(m0, th, tw);
    const int nrows = pin(min(m0 + BM, mlim) - 1, th, tw) + (R - 1) * Wi + S - ps;   // <= PR (host-checked)

    // per 32-pixel block of this lane: its panel row at tap (0,0), and one bit per tap that falls inside the image
    int prow[MB];
    unsigned inside[MB];
#pragma unroll
    for (int bm = 0; bm < MB; bm++) {
        const int m = m0 + (wm * MB + bm) * 32 + li;
        prow[bm] = 0;
        inside[bm] = 0u;
        if (m < mlim) {
            int hh, ww;
            prow[bm] = pin(m, hh, ww) - ps;
            for (int r = 0, tap = 0; r < R; r++)
                for (int s = 0; s < S; s++, tap++)
                    if ((unsigned)(hh + r) < (unsigned)Hi && (unsigned)(ww + s) < (unsigned)Wi) inside[bm] |= 1u << tap;
        }
    }

    // ---- panel loader: thread -> (row, 8-channel half) pairs u = tid + i * NT.  Rows before the first or past the last
    // pixel of the tensor and rows the tile does not need get an offset outside the descriptor and read as zeros.
    const unsigned in_bytes = LOAD == XC_BLOCKS ? (unsigned)(p.g.N * p.g.H * p.g.W) * (unsigned)p.g.C * 4u
                                                : (unsigned)(p.g.N * Hi * Wi) * (unsigned)Cred * 4u;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(p.a, in_bytes);
    const __amdgpu_buffer_rsrc_t mrs = owt_make_rsrc(MASKED ? p.mask : p.a, in_bytes);
    unsigned rowoff[PU];                             // byte offset of the row's first value
    unsigned out_bits[LOAD == XC_BLOCKS ? PU : 1];   // blocks: bit dy * sw + dx is set where that pixel lies outside the image
#pragma unroll
    for (int i = 0; i < PU; i++) {
        const int u = tid + i * NT, row = u >> 1, pix = ps + row;
        const bool there = row < nrows && (unsigned)pix < (unsigned)(p.g.N * Hi * Wi);
        if (LOAD == XC_BLOCKS) {
            const int n = p.dHpWp.div(pix), rem = pix - n * (Hi * Wi), by = p.dWp.div(rem), bx = rem - by * Wi;
            const int y0 = by * p.g.sh - p.g.ph, x0 = bx * p.g.sw - p.g.pw;
            unsigned bits = 0xffffffffu;
            if (there)
                for (int dy = 0, q = 0; dy < p.g.sh; dy++)
                    for (int dx = 0; dx < p.g.sw; dx++, q++)
                        if ((unsigned)(y0 + dy) < (unsigned)p.g.H && (unsigned)(x0 + dx) < (unsigned)p.g.W) bits &= ~(1u << q);
            out_bits[LOAD == XC_BLOCKS ? i : 0] = bits;
            rowoff[i] = (unsigned)(((n * p.g.H + y0) * p.g.W + x0) * p.g.C) * 4u;
        } else {
            rowoff[i] = there ? (unsigned)pix * (unsigned)Cred * 4u : OOB;
        }
    }
    // blocks: where value c of a block is: byte offset from its first pixel, and 31 - its pixel's bit
    constexpr int CTAB = LOAD == XC_BLOCKS ? 256 : 1;
    __shared__ uint2 ctab[CTAB];
    if (LOAD == XC_BLOCKS) {
        const int rowc = p.g.sw * p.g.C;
        for (int c = tid; c < p.ksteps * 16; c += NT) {
            const int dy = c / rowc, rem = c - dy * rowc;
            // values past the block read as zeros: the offset alone puts them outside the descriptor
            ctab[c] = dy < p.g.sh ? make_uint2((unsigned)((dy * p.g.W * p.g.C + rem) * 4), (unsigned)(31 - (dy * p.g.sw + rem / p.g.C)))
                                  : make_uint2(OOB, 0u);
        }
        __syncthreads();
    }
    float preg[PU][8], yreg[MASKED ? PU : 1][8];
    auto load8 = [&](__amdgpu_buffer_rsrc_t rs, unsigned base, int c, float (&v)[8]) __attribute__((always_inline)) {
        if (LOAD == XC_VEC) {
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const float4 f = buffer_load4(rs, c + 4 * q < Cred ? base + (unsigned)(c + 4 * q) * 4u : OOB);
                v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
                v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(c + j < Cred ? base + (unsigned)(c + j) * 4u : OOB), 0, 0));
        }
    };
    auto load_blocks = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const uint2 at = ctab[LOAD == XC_BLOCKS ? ch * 16 + (tid & 1) * 8 + j : 0];
#pragma unroll
            for (int i = 0; i < PU; i++) {
                const unsigned off = (rowoff[i] + at.x) | ((out_bits[LOAD == XC_BLOCKS ? i : 0] << at.y) & OOB);
                preg[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ars, (int)(at.x == OOB ? OOB : off), 0, 0));
            }
        }
    };
    auto load_panel = [&](int ch) __attribute__((always_inline)) {
        if (LOAD == XC_BLOCKS) { load_blocks(ch); return; }
        const int c = ch * 16 + (tid & 1) * 8;
#pragma unroll
        for (int i = 0; i < PU; i++) {
            load8(ars, rowoff[i], c, preg[i]);
            if (MASKED) load8(mrs, rowoff[i], c, yreg[MASKED ? i : 0]);
        }
    };
    auto store_panel = [&](uint4 *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PU; i++) {
            const int u = tid + i * NT, row = u >> 1, half = u & 1;
            if (MASKED) {
#pragma unroll
                for (int j = 0; j < 8; j++) preg[i][j] = yreg[MASKED ? i : 0][j] > 0.f ? preg[i][j] : 0.f;
            }
            uint4 h, m, l;
            split3_scaled(preg[i], h, m, l);
            if (row < PR) {
                uint4 *q = dst + half * PL + row;
                q[0] = h; q[2 * PL] = m; q[4 * PL] = l;
            }
        }
    };

    // ---- filter slices: SL pieces of 1 KB, dealt to the wavefronts in turn
    const int nblocks = p.tiles_n * (BN / 32);
    const owt_i32x4 brs = make_rsrc(p.b, (unsigned)(p.ksteps * RS * nblocks) * 3072u);
    const unsigned slice_lds = (unsigned)(size_t)(__attribute__((address_space(3))) uint4 *)slices;
    const unsigned bpiece = (unsigned)(tn * (BN / 32)) * 3072u + (unsigned)wave * 1024u + (unsigned)lane * 16u;
    constexpr int SQ = SL / NW, SREM = SL % NW;                      // pieces per wavefront: SQ, one more for the first SREM
    auto fetch_slice = [&](int ch, int tap, int slot) __attribute__((always_inline)) {
        const unsigned off = bpiece + (unsigned)((ch * RS + tap) * nblocks) * 3072u;
        const unsigned dst = slice_lds + (unsigned)(slot * SL + wave) * 1024u;
#pragma unroll
        for (int i = 0; i < SQ; i++) buffer_load16_to_lds(brs, off + (unsigned)(i * NW) * 1024u, dst + (unsigned)(i * NW) * 1024u);
        if (SREM && wave < SREM) buffer_load16_to_lds(brs, off + (unsigned)(SQ * NW) * 1024u, dst + (unsigned)(SQ * NW) * 1024u);
    };
    // This wavefront's slice pieces have landed, except those of the slice requested last (`younger`) and the panel loads
    // requested before it (`panel_too`); then the work-group meets.  Fragment reads stay in flight across the barrier: what
    // is overwritten after it was read before the previous one.
    // (Only 16-byte panel loads are counted: two smaller ones could become one in the compiler's hands.)
    constexpr int NPL = LOAD == XC_VEC ? PU * 2 * (MASKED ? 2 : 1) : 0;        // panel loads per thread
    auto meet = [&](bool younger, bool panel_too) __attribute__((always_inline)) {
        if (!younger) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        else if (NPL > 0 && NPL + SQ + 1 <= 63 && panel_too) {
            if (SREM && wave < SREM) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((NPL + SQ + 1) & 63) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((NPL + SQ) & 63) : "memory");
        } else if (SREM && wave < SREM) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(SQ + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(SQ) : "memory");
    };

    split_acc big[MB][2], small[MB][2];
#pragma unroll
    for (int i = 0; i < MB; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) big[i][j][r] = small[i][j][r] = 0.f;

    if (tid < 6) panel[tid * PL + PR] = make_uint4(0u, 0u, 0u, 0u);           // the row of zeros of every plane
    const int nsteps = (ch_end - ch_beg) * RS;                                // one step per (chunk, tap); at least one
    load_panel(ch_beg);
    store_panel(panel);
    auto next_step = [&](int &c, int &t) { if (++t == RS) { t = 0; c++; } };
    int ch3 = ch_beg, tap3 = 0;                                               // the next slice to request
    for (int i = 0; i < 3 && i < nsteps; i++) { fetch_slice(ch3, tap3, i); next_step(ch3, tap3); }

    // The fragments of a step are read during the step before it, each right behind the last product that needs its old
    // value: parts of a step, in the order of their last use, l of the pixels, l of the filters, m, m, h, h.
    split_frag a[MB][3], f[2][3];
    const uint4 *arow[MB], *bp;
    auto aim = [&](int tap, int r, int s, int slot) __attribute__((always_inline)) {
        const int shift = r * Wi + s;
#pragma unroll
        for (int bm = 0; bm < MB; bm++) arow[bm] = panel + lh * PL + (((inside[bm] >> tap) & 1u) ? prow[bm] + shift : PR);
        bp = slices + (slot * SL + wn * 6) * 64 + lane;
    };
    auto read_a = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int bm = 0; bm < MB; bm++) a[bm][q] = __builtin_bit_cast(split_frag, arow[bm][2 * q * PL]);
    };
    auto read_b = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int bn = 0; bn < 2; bn++) f[bn][q] = __builtin_bit_cast(split_frag, bp[(bn * 3 + q) * 64]);
    };
    auto product = [&](int qa, int qb) __attribute__((always_inline)) {
#pragma unroll
        for (int bm = 0; bm < MB; bm++)
#pragma unroll
            for (int bn = 0; bn < 2; bn++) {
                split_acc &acc = qa + qb == 0 ? big[bm][bn] : small[bm][bn];
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[bm][qa], f[bn][qb], acc, 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };

    // slices 0 and 1 have landed (meet() leaves the youngest in flight), the panel is written
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    meet(nsteps > 2, false);
    aim(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 3; q++) { read_a(q); read_b(q); }
    // A step begins with the meeting that says the next step's slice has landed, and requests the slice three steps ahead into
    // the slot of the step before it.  A chunk's first step requests the next chunk's panel in between (held in registers
    // until the last tap), so its loads have two steps' time before a meeting waits for them.
    int t = 0, slot = 0;
    auto begin = [&](int load, bool panel_too) __attribute__((always_inline)) {
        if (t > 0) meet(t + 2 < nsteps, panel_too);
        if (load < ch_end) load_panel(load);
        if (t + 3 < nsteps) { fetch_slice(ch3, tap3, slot == 0 ? 3 : slot - 1); next_step(ch3, tap3); }
        slot = slot == 3 ? 0 : slot + 1;
        t++;
    };
    for (int ch = ch_beg; ch < ch_end; ch++) {
        for (int tap = 1, r = 0, s = 0; tap < RS; tap++) {                    // the step of tap - 1
            begin(tap == 1 ? ch + 1 : ch_end, tap == 2 && ch + 1 < ch_end);
            if (++s == S) { s = 0; r++; }
            aim(tap, r, s, slot);
            product(1, 1);
            product(2, 0); read_a(2);
            product(0, 2); read_b(2);
            product(1, 0); read_a(1);
            product(0, 1); read_b(1);
            product(0, 0); read_a(0); read_b(0);
        }
        begin(RS == 1 ? ch + 1 : ch_end, false);                              // the last tap
        product(1, 1); product(2, 0); product(0, 2); product(1, 0); product(0, 1); product(0, 0);
        if (ch + 1 < ch_end) {
            asm volatile("s_barrier" ::: "memory");                           // everyone has its fragments of the old panel
            store_panel(panel);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            aim(0, 0, 0, slot);
#pragma unroll
            for (int q = 0; q < 3; q++) { read_a(q); read_b(q); }
        }
    }

    // ---- epilogue: register r of lane (li, lh) of block (bm, bn) is pixel 8*(r/4) + 4*lh + r%4, column li.  Columns past
    // the end and pixels past the last get an offset outside the descriptor: their stores are dropped.
    // (the lane's place is worked out anew: kept over the loop, it is spilled where registers are short)
    const int elane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), eli = elane & 31, elh = elane >> 5;
    const bool part = p.splits > 1;
    const unsigned out_bytes = (unsigned)mlim * (unsigned)p.Ncols * 4u;
    const __amdgpu_buffer_rsrc_t ors = owt_make_rsrc(part ? (const void *)(p.partial + (size_t)split * p.M * p.Ncols) : p.out, out_bytes);
    const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(BWD && p.xmask ? p.xmask : p.a, BWD && p.xmask ? out_bytes : 0u);
    const bool xm = BWD && !part && p.xmask != nullptr;
    auto rowstep = [&](int q) { return (unsigned)(8 * (q / 4) + q % 4) * (unsigned)p.Ncols * 4u; };   // an offset past OOB stays past it
    const bool relu = !BWD && !part && (p.flags & 2u);
    float sum = 0.f;                                                          // not finite if an output may have to be worked out again
#pragma unroll
    for (int bn = 0; bn < 2; bn++) {
        const int n = n0 + wn * 64 + bn * 32 + eli;
        const float bias = (!BWD && !part && (p.flags & 1u) && n < p.Ncols) ? p.bias[n] : 0.f;
#pragma unroll
        for (int bm = 0; bm < MB; bm++) {
            const unsigned m = (unsigned)(m0 + (wm * MB + bm) * 32 + 4 * elh);
            const unsigned base = n < p.Ncols ? (m * (unsigned)p.Ncols + (unsigned)n) * 4u : OOB;
            float x[16];
            if (xm) {
#pragma unroll
                for (int q = 0; q < 16; q++)
                    x[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrs, (int)(base + rowstep(q)), 0, 0));
            }
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const float t = big[bm][bn][q] + small[bm][bn][q];
                sum += LOAD == XC_BLOCKS ? t : big[bm][bn][q];
                float v = t * kSplitUnscale + bias;
                if (relu) v = v > 0.f ? v : 0.f;
                if (xm) v = x[q] > 0.f ? v : 0.f;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ors, (int)(base + rowstep(q)), 0, 0);
            }
        }
    }

    // Outputs worked out again, each lane its own, one multiply-add at a time and only until the sum is NaN (which it then
    // stays), and stored over the first result:
    //  * those whose large products left the range of the scaled operands (a sum past 2^80, a value past 2^104).  Infinities and
    //    NaN among the operands leave the large products finite (split3_scaled) and are right as they are;
    //  * a block of a strided pass holds pixels outside the window, met by zero filter values: an infinity or NaN among them
    //    reaches the sum, so there it is every output that is not finite.
    if (__ballot(!(fabsf(sum) < __builtin_inff())) != 0) {
        unsigned long long redo = 0;                                          // bit 32 * bm + 16 * bn + q
#pragma unroll
        for (int i = 0; i < MB * 32; i++) {
            const float t = big[i >> 5][(i >> 4) & 1][i & 15] + (LOAD == XC_BLOCKS ? small[i >> 5][(i >> 4) & 1][i & 15] : 0.f);
            if (!(fabsf(t) < __builtin_inff())) redo |= 1ull << i;
        }
        const float *x = (const float *)p.a, *y = (const float *)p.mask, *w = (const float *)p.b0;
        const Geom &g = p.g;
        const int kd_beg = ch_beg * 16, kd_end = ch_end * 16;                 // this split's part of the reduction
        for (; redo; redo &= redo - 1) {
            const int i = __ffsll(redo) - 1;
            const int m = m0 + (wm * MB + (i >> 5)) * 32 + 8 * ((i & 15) / 4) + 4 * elh + i % 4, n = n0 + wn * 64 + ((i >> 4) & 1) * 32 + eli;
            if (m >= mlim || n >= p.Ncols) continue;
            const int im = p.dHoWo.div(m), rem = m - im * HoWo, po = p.dWo.div(rem), qo = rem - po * p.Wo;
            float v = 0.f;
            if (LOAD == XC_BLOCKS) {
                for (int r2 = 0, dy = 0; r2 < p.R0 && v == v; r2++, dy = dy + 1 == g.sh ? 0 : dy + 1) {
                    const int hh = po * g.sh - g.ph + r2;
                    for (int s2 = 0, dx = 0; s2 < p.S0 && v == v; s2++, dx = dx + 1 == g.sw ? 0 : dx + 1) {
                        const int ww = qo * g.sw - g.pw + s2, kd = (dy * g.sw + dx) * g.C;
                        const bool in = (unsigned)hh < (unsigned)g.H && (unsigned)ww < (unsigned)g.W;
                        const float *xp = x + ((size_t)(im * g.H + (in ? hh : 0)) * g.W + (in ? ww : 0)) * g.C;
                        const float *wp = w + ((size_t)(n * p.R0 + r2) * p.S0 + s2) * g.C;
                        for (int c = max(0, kd_beg - kd); c < min(g.C, kd_end - kd); c++) v = fmaf(in ? xp[c] : 0.f, wp[c], v);
                    }
                }
            } else {
                for (int tap = 0, r = 0, s = 0; tap < RS && v == v; tap++) {
                    const int hh = po - p.pah + r, ww = qo - p.paw + s;
                    const bool in = (unsigned)hh < (unsigned)Hi && (unsigned)ww < (unsigned)Wi;
                    const size_t at = ((size_t)(im * Hi + (in ? hh : 0)) * Wi + (in ? ww : 0)) * Cred;
                    // forward: w[n][tap][c]; backward-data: w[c][RS-1-tap][n]
                    const float *wp = w + (BWD ? (size_t)(RS - 1 - tap) * p.Ncols + n : ((size_t)n * RS + tap) * Cred);
                    const size_t step = BWD ? (size_t)RS * p.Ncols : 1;
                    for (int c = kd_beg; c < min(Cred, kd_end); c++)
                        v = fmaf(in && (!MASKED || y[at + c] > 0.f) ? x[at + c] : 0.f, wp[c * step], v);
                    if (++s == S) { s = 0; r++; }
                }
            }
            if (!part) {
                if (!BWD && (p.flags & 1u)) v += p.bias[n];
                if (relu) v = v > 0.f ? v : 0.f;
                if (xm && !(((const float *)p.xmask)[(size_t)m * p.Ncols + n] > 0.f)) v = 0.f;
            }
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ors, (int)(((unsigned)m * (unsigned)p.Ncols + (unsigned)n) * 4u), 0, 0);
        }
    }
}

}  // namespace owt
