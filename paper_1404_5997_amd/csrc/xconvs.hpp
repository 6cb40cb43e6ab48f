// Direct stride-1 convolution, fp32 storage, operands split in three (split3.hpp), for layers of few tiles: forward and
// backward-data (Section 4 of the paper, forward step 2 / backward step 2).
//
// With a work-group or less per CU xconv.hpp is a chain of latencies: a launch that lays out the filters, then one tap after the
// other, each behind a barrier, with one wavefront per SIMD and nothing beside it (25 taps of an 8-image 32x32x3 layer: 15 us for
// 1.2 us of products).  Here
//  * a work-group is TG groups of WM wavefronts; the groups share the panel and take every TG-th tap, so their latencies
//    overlap, and add up through LDS in a fixed order at the end (no partial sums in memory, no reduce pass);
//  * a wavefront loads its filter fragments from the filters as they are, two steps ahead, and splits them itself: no
//    launch before, no scratch, no slice in LDS and no barrier but the two that change the panel;
//  * a wavefront owns 32 pixels x 32 filters, so layers of few filters waste less.
//  * a panel holds as many 16-channel chunks as leave a thread one piece of it to load (two or three of the smallest panels): the
//    groups share 18 taps, not 9, and barriers halve.  37 images 15x11, 100 -> 72 22.3 -> 20.3 us forward, 22.6 -> 20.1 backward-data;
//    50 drawn layers 2 and 3 % on average.
// Splitting filters per wavefront is 56 vector instructions a fragment (of 6 matrix instructions), which is why layers that fill the
// chip stay with xconv.hpp; the planner's cost model draws the line.
//
// Measured against xconv.hpp with its layout launch: 8 images of 32x32x3 to 16 filters of 5x5 17.6 -> 7.2 us forward, 17.5 -> 7.9 us
// backward-data; 37 of 15x11x100 to 72 of 3x3 25.3 -> 21.8; one 53x31x32 image to 66 of 5x5 43.9 -> 17.3; 120 passes of 60 layers
// under 14 GFLOP 3287 -> 2701 us together.  What is left is latency: first loads, a tap's panel reads, split and matrix instructions one
// behind the other (367 clocks), the stores.
#pragma once
#include "igemm.hpp"
#include "owt_host.hpp"
#include "split3.hpp"

namespace owt {

// VEC: panel values 16 bytes at a time (reduction channels a multiple of four).  R * S >= TG (host-checked), at most 32 taps; 32-bit byte
// offsets in every tensor (host-checked).
template <bool BWD, int WM, int TG, int PR, bool VEC, bool MASKED>
__global__ void __launch_bounds__(64 * WM * TG, TG == 8 ? 2 : 4) xconvs_kernel(const GemmParams p)
{
    constexpr int NT = 64 * WM * TG, BM = 32 * WM;
    constexpr int CH = xconvs_chunks(WM, TG, PR), PC = 2 * CH;                        // 16-channel chunks in a panel, and pieces of 8 channels of a row
    constexpr int PL = PR + 1, PANEL = 6 * CH * PL, RED = TG * WM * 256;              // 16-byte units
    constexpr int PU = (PC * PR + NT - 1) / NT;
    constexpr unsigned OOB = 0x80000000u;

    // the groups' sums; the panel, in the same place unless each wavefront's sums put by (its own 16 bytes a lane, four times) are in the first
    constexpr bool PUT_LDS = MASKED && PU > 1;                                       // (16 more registers would not fit)
    __shared__ __attribute__((aligned(16))) uint4 lds[PUT_LDS ? RED + PANEL : PANEL > RED ? PANEL : RED];
    uint4 *panel = lds + (PUT_LDS ? RED : 0);
    float *red = (float *)lds;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5, wm = wave % WM, grp = wave / WM;

    const int ntiles = p.tiles_m * p.tiles_n;
    const int b = blockIdx.x, xcd = b & 7;
    const int logical = xcd * (ntiles >> 3) + min(xcd, ntiles & 7) + (b >> 3);
    const int tm = logical / p.tiles_n, tn = logical - tm * p.tiles_n;
    const int m0 = tm * BM, n0 = tn * 32, split = blockIdx.y;
    const int ch_beg = split * p.ksteps_per_split, ch_end = min(p.ksteps, ch_beg + p.ksteps_per_split);

    const int R = p.g.R, S = p.g.S, RS = R * S, Hi = p.Hi, Wi = p.Wi, Cred = p.Cred, HoWo = p.Ho * p.Wo;
    auto pin = [&](int m, int &hh, int &ww) {
        const int n = p.dHoWo.div(m), rem = m - n * HoWo;
        const int ho = p.dWo.div(rem), wo = rem - ho * p.Wo;
        hh = ho - p.pah; ww = wo - p.paw;
        return n * Hi * Wi + hh * Wi + ww;
    };
    int hh, ww;
    const int ps = pin(m0, hh, ww);
    const int nrows = pin(min(m0 + BM, p.M) - 1, hh, ww) + (R - 1) * Wi + S - ps;    // <= PR (host-checked)

    // this lane's panel row at tap (0,0), and one bit per tap that falls inside the image
    int prow = 0;
    unsigned inside = 0u;
    {
        const int m = m0 + wm * 32 + li;
        if (m < p.M) {
            prow = pin(m, hh, ww) - ps;
            for (int r = 0, tap = 0; r < R; r++)
                for (int s = 0; s < S; s++, tap++)
                    if ((unsigned)(hh + r) < (unsigned)Hi && (unsigned)(ww + s) < (unsigned)Wi) inside |= 1u << tap;
        }
    }

    // ---- panel: thread -> (row, piece of eight channels) pairs u = tid + i * NT, as in xconv.hpp
    const unsigned in_bytes = (unsigned)(p.g.N * Hi * Wi) * (unsigned)Cred * 4u;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(p.a, in_bytes), mrs = owt_make_rsrc(MASKED ? p.mask : p.a, in_bytes);
    unsigned rowoff[PU];
#pragma unroll
    for (int i = 0; i < PU; i++) {
        const int u = tid + i * NT, row = u / PC, pix = ps + row;
        rowoff[i] = row < nrows && (unsigned)pix < (unsigned)(p.g.N * Hi * Wi) ? (unsigned)pix * (unsigned)Cred * 4u : OOB;
    }
    float preg[PU][8], yreg[MASKED ? PU : 1][8];
    auto load8 = [&](__amdgpu_buffer_rsrc_t rs, unsigned base, int c, float (&v)[8]) __attribute__((always_inline)) {
        if (VEC) {
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
    auto load_panel = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PU; i++) {
            const int c = ch * 16 + (tid + i * NT) % PC * 8;
            load8(ars, rowoff[i], c, preg[i]);
            if (MASKED) load8(mrs, rowoff[i], c, yreg[MASKED ? i : 0]);
        }
    };
    auto store_panel = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PU; i++) {
            const int u = tid + i * NT, row = u / PC, piece = u % PC;
            if (MASKED) {
#pragma unroll
                for (int j = 0; j < 8; j++) preg[i][j] = yreg[MASKED ? i : 0][j] > 0.f ? preg[i][j] : 0.f;
            }
            uint4 h, m, l;
            split3_scaled(preg[i], h, m, l);
            if (row < PR) {
                uint4 *q = panel + (piece / 2 * 6 + piece % 2) * PL + row;
                q[0] = h; q[2 * PL] = m; q[4 * PL] = l;
            }
        }
    };

    // ---- filters: this lane's column, eight reduction values of a tap.  Forward: w[n][tap][c], contiguous.  Backward-data:
    // w[c][RS-1-tap][n].  What lies past the reduction or the last column reads as zeros.
    const __amdgpu_buffer_rsrc_t brs = owt_make_rsrc(p.b, (unsigned)p.Ncols * (unsigned)Cred * (unsigned)RS * 4u);
    const int n = n0 + li;
    const unsigned bcol = n < p.Ncols ? (BWD ? (unsigned)n * 4u : (unsigned)n * (unsigned)(RS * Cred) * 4u) : OOB;
    float braw[2][8];
    auto load_b = [&](int ch, int tap, int u) __attribute__((always_inline)) {
        const int c = ch * 16 + 8 * lh;
        if (BWD) {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const unsigned at = bcol + (unsigned)((c + j) * RS + (RS - 1 - tap)) * (unsigned)p.Ncols * 4u;
                braw[u][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(brs, (int)(c + j < Cred && bcol != OOB ? at : OOB), 0, 0));
            }
        } else {
            const unsigned at = bcol + (unsigned)(tap * Cred + c) * 4u;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const float4 f = buffer_load4(brs, bcol != OOB && c + 4 * q < Cred ? at + 16u * q : OOB);
                braw[u][4 * q] = f.x; braw[u][4 * q + 1] = f.y; braw[u][4 * q + 2] = f.z; braw[u][4 * q + 3] = f.w;
            }
        }
    };

    split_acc big, small;
#pragma unroll
    for (int q = 0; q < 16; q++) big[q] = small[q] = 0.f;

    if (tid < 6 * CH) panel[tid * PL + PR] = make_uint4(0u, 0u, 0u, 0u);      // the row of zeros of every plane
    // A panel's steps are its chunks' taps one after the other, and this group's are grp, grp + TG, ...: (chunk in the panel, tap)
    struct Step { int ch0, k, tap; };
    auto advance = [&](Step &a) __attribute__((always_inline)) {
        a.tap += TG;
        if (CH == 1) {
            if (a.tap >= RS) { a.tap = grp; a.ch0++; }
            return;
        }
        if (a.tap >= RS) { a.tap -= RS; a.k++; }                              // (TG <= RS)
        if (a.k >= min(CH, ch_end - a.ch0)) { a.ch0 += CH; a.k = 0; a.tap = grp; }
    };
    auto steps_of = [&](int chunks) { return (chunks * RS - grp + TG - 1) / TG; };
    const int nch = ch_end - ch_beg, nsteps = nch / CH * steps_of(CH) + (nch % CH ? steps_of(nch % CH) : 0);
    Step ld = {ch_beg, 0, grp};                                               // the step whose filters are loaded next
    auto load_next = [&](int u) __attribute__((always_inline)) {
        if (ld.ch0 < ch_end) load_b(ld.ch0 + (CH > 1 ? ld.k : 0), ld.tap, u);
        advance(ld);
    };
    load_panel(ch_beg);
    load_next(0);
    load_next(1);
    // A chain of n instructions rounds off more the longer it is, and layers that come here from many splits of xconv.hpp had short ones
    // there.  So the high parts' sums are put by at the first change of panel after kRun steps, and those sums added up.  Error of y
    // against 64 bits, xconv.hpp, one chain, this: 5 images 20x12, 224 -> 383 of 3x3 9.1e-8, 1.10e-7, 8.3e-8; 12 of 26x35, 128 -> 19 7.8e-8, 8.9e-8,
    // 7.8e-8; none of 320 passes is off by more than with xconv.hpp now, 7 of 140 were.  After 12 steps one pass is off by 2 % more.  The sums in LDS
    // instead of 16 registers: 180 passes of drawn layers 5043 us instead of 5001.
    constexpr int kRun = 10;
    float4 *mine = (float4 *)lds + wave * 256 + lane;
    split_acc total;
#pragma unroll
    for (int q = 0; q < 16; q++) total[q] = 0.f;
    int since = 0;
    bool put = false;
    auto put_by = [&]() __attribute__((always_inline)) {
        if (PUT_LDS) {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                float4 t = put ? mine[64 * q] : make_float4(0.f, 0.f, 0.f, 0.f);
                t.x += big[4 * q]; t.y += big[4 * q + 1]; t.z += big[4 * q + 2]; t.w += big[4 * q + 3];
                mine[64 * q] = t;
            }
            put = true;
        }
#pragma unroll
        for (int q = 0; q < 16; q++) {
            if (!PUT_LDS) total[q] += big[q];
            big[q] = 0.f;
        }
        since = 0;
    };
    Step at = {ch_beg, 0, grp};
    bool fresh = true;                                                        // the step is the first of its panel
    for (int i = 0; i < nsteps; i += 2) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            if (i + u >= nsteps) break;
            const int k = CH > 1 ? at.k : 0, ch = at.ch0 + k, tap = at.tap;
            if (fresh) {                                                      // a new panel; every wavefront comes here once a panel
                if (at.ch0 > ch_beg) __syncthreads();                         // everyone has its fragments of the old panel
                store_panel();
                if (since + (CH > 1 ? steps_of(min(CH, ch_end - at.ch0)) - 3 : 0) >= kRun) put_by();
                __syncthreads();
                if (at.ch0 + CH < ch_end) load_panel(at.ch0 + CH);
            }
            since++;
            const int r = p.g.dS.div(tap), s = tap - r * S;
            const uint4 *arow = panel + (k * 6 + lh) * PL + (((inside >> tap) & 1u) ? prow + r * Wi + s : PR);
            split_frag a[3], f[3];
#pragma unroll
            for (int q = 0; q < 3; q++) a[q] = __builtin_bit_cast(split_frag, arow[2 * q * PL]);
            const int left = Cred - (ch * 16 + 8 * lh);                       // reduction values of this lane's eight that exist
            if (!BWD && ch * 16 + 16 > Cred) {                                // what follows a tap's channels belongs to the next tap
#pragma unroll
                for (int j = 0; j < 8; j++) braw[u][j] = j < left ? braw[u][j] : 0.f;
            }
            uint4 h, m, l;
            split3_scaled(braw[u], h, m, l);
            f[0] = __builtin_bit_cast(split_frag, h); f[1] = __builtin_bit_cast(split_frag, m); f[2] = __builtin_bit_cast(split_frag, l);
            load_next(u);
            constexpr int PA[6] = {1, 2, 0, 1, 0, 0}, PB[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
            for (int e = 0; e < 6; e++) {
                split_acc &acc = e == 5 ? big : small;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[e]], f[PB[e]], acc, 0, 0, 0);
            }
            const int ch0 = at.ch0;
            advance(at);
            fresh = at.ch0 != ch0;
        }
    }

    // ---- the groups' sums, in pairs.  Every wavefront adds up 16 / TG of the registers, first of the high parts'
    // products and then of the others: the first are nearly exact as long as they stand by themselves (16-bit products in a
    // 24-bit sum), and with the two added in each group already y of the 75-term layer above was 1.3 times as far from 64 bits.
    constexpr int QN = 16 / TG;
    const int q0 = grp * QN;
    float v[QN];
    if (PUT_LDS && put) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const float4 t = mine[64 * q];
            total[4 * q] = t.x; total[4 * q + 1] = t.y; total[4 * q + 2] = t.z; total[4 * q + 3] = t.w;
        }
    }
#pragma unroll
    for (int q = 0; q < 16; q++) big[q] += total[q];
#pragma unroll
    for (int half = 0; half < 2; half++) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; q++) red[(grp * WM + wm) * 1024 + q * 64 + lane] = half ? small[q] : big[q];
        __syncthreads();
        float t[QN];
#pragma unroll
        for (int j = 0; j < QN; j++) {
            float g[TG];
#pragma unroll
            for (int k = 0; k < TG; k++) g[k] = red[(k * WM + wm) * 1024 + (q0 + j) * 64 + lane];
#pragma unroll
            for (int d = 1; d < TG; d *= 2)                                  // (one chain of eight rounds off more)
#pragma unroll
                for (int k = 0; k < TG; k += 2 * d) g[k] += g[k + d];
            t[j] = g[0];
            v[j] = half ? v[j] + t[j] : t[j];
        }
    }

    // ---- epilogue: register q of lane (li, lh) is pixel 8*(q/4) + 4*lh + q%4, column li.  Columns and pixels past the end get an offset
    // outside the descriptor: their stores are dropped.
    const bool part = p.splits > 1, relu = !BWD && !part && (p.flags & 2u), xm = BWD && !part && p.xmask != nullptr;
    const unsigned out_bytes = (unsigned)p.M * (unsigned)p.Ncols * 4u;
    const __amdgpu_buffer_rsrc_t ors = owt_make_rsrc(part ? (const void *)(p.partial + (size_t)split * p.M * p.Ncols) : p.out, out_bytes);
    const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(BWD && p.xmask ? p.xmask : p.a, BWD && p.xmask ? out_bytes : 0u);
    const int mq = m0 + wm * 32 + 8 * (q0 / 4) + 4 * lh + q0 % 4;
    const float bias = (!BWD && !part && (p.flags & 1u) && n < p.Ncols) ? p.bias[n] : 0.f;
    const unsigned base = n < p.Ncols ? ((unsigned)mq * (unsigned)p.Ncols + (unsigned)n) * 4u : OOB;
    float x[QN];
    if (xm) {
#pragma unroll
        for (int j = 0; j < QN; j++) x[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrs, (int)(base + (unsigned)j * (unsigned)p.Ncols * 4u), 0, 0));
    }
    unsigned redo = 0;
#pragma unroll
    for (int j = 0; j < QN; j++) {
        if (!(fabsf(v[j]) < __builtin_inff())) redo |= 1u << j;
        float o = v[j] * kSplitUnscale + bias;
        if (relu) o = o > 0.f ? o : 0.f;
        if (xm) o = x[j] > 0.f ? o : 0.f;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ors, (int)(base + (unsigned)j * (unsigned)p.Ncols * 4u), 0, 0);
    }

    // Outputs that are not finite, each lane its own, worked out again one multiply-add at a time and only until the sum is NaN,
    // and stored over the first result: a sum may have left the range of the scaled operands (split3_scaled), and one that an
    // infinity or a NaN among the operands made comes out the same.
    if (__ballot(redo != 0) != 0) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                                   // vmcnt(0): the first results are stored
        const float *xs = (const float *)p.a, *ys = (const float *)p.mask, *w = (const float *)p.b;
        for (; redo; redo &= redo - 1) {
            const int m = mq + __ffs(redo) - 1;
            if (m >= p.M || n >= p.Ncols) continue;
            const int im = p.dHoWo.div(m), rem = m - im * HoWo, po = p.dWo.div(rem), qo = rem - po * p.Wo;
            float o = 0.f;
            for (int t = 0, r = 0, s = 0; t < RS && o == o; t++) {
                const int h2 = po - p.pah + r, w2 = qo - p.paw + s;
                const bool in = (unsigned)h2 < (unsigned)Hi && (unsigned)w2 < (unsigned)Wi;
                const size_t at = ((size_t)(im * Hi + (in ? h2 : 0)) * Wi + (in ? w2 : 0)) * Cred;
                const float *wp = w + (BWD ? (size_t)(RS - 1 - t) * p.Ncols + n : ((size_t)n * RS + t) * Cred);
                const size_t step = BWD ? (size_t)RS * p.Ncols : 1;
                for (int c = ch_beg * 16; c < min(Cred, ch_end * 16); c++)
                    o = fmaf(in && (!MASKED || ys[at + c] > 0.f) ? xs[at + c] : 0.f, wp[c * step], o);
                if (++s == S) { s = 0; r++; }
            }
            if (!part) {
                if (!BWD && (p.flags & 1u)) o += bias;
                if (relu) o = o > 0.f ? o : 0.f;
                if (xm && !(((const float *)p.xmask)[(size_t)m * p.Ncols + n] > 0.f)) o = 0.f;
            }
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ors, (int)(((unsigned)m * (unsigned)p.Ncols + (unsigned)n) * 4u), 0, 0);
        }
    }
}

}  // namespace owt
