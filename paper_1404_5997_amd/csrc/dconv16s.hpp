// Direct stride-1 convolution, bf16 storage, for layers of few tiles: forward and backward-data (Section 4 of the paper, forward
// step 2 / backward step 2).
//
// With a work-group or less per CU the kernels of dconv_bf16p.hpp are a chain of latencies: a launch that lays out the filters, then
// 64 to 128 pixels a wavefront, one tap after the other behind barriers (0.7 us a tap, 14 to 30 us for layers of a few
// microseconds' work).  As in xconvs.hpp a work-group is TG groups of WM wavefronts that share the panel, take every TG-th tap and add up
// through LDS in a fixed order at the end; a wavefront owns 32 pixels x 32 filters and loads its filter fragments from the
// filters as they are, two steps ahead: no launch before, and no barrier but the two that change the panel.  Every wavefront
// loads its own filters, which is why layers that fill the chip stay with the other kernels; the planner's cost model draws the line.
//
// Measured against those kernels, us: 3 images 7x19, 160 -> 43 channels of 3x3 22.1 -> 7.5 forward, 19.3 -> 9.3 backward-data; 4 of 6x52,
// 32 -> 172 of 5x5 26.2 -> 6.2 and 25.7 -> 15.3; of 110 drawn layers under 15 GFLOP it takes 79 passes,
// 1553 -> 812 (all 220 5304 -> 4548).  What is left is latency: a
// step's panel reads and filter loads (150 clocks and 36 a load).
#pragma once
#include "dconv_bf16.hpp"

namespace owt {

// E: elements a load may take at once (8, 2 or 1: reduction channels a multiple of it).  R * S >= TG (host-checked), at most 32 taps;
// 32-bit byte offsets in every tensor (host-checked).
template <bool BWD, int WM, int TG, int PR, int E, bool MASKED>
__global__ void __launch_bounds__(64 * WM * TG, TG == 8 ? 2 : 4) dconv16s_kernel(const GemmParams p)
{
    constexpr int NT = 64 * WM * TG, BM = 32 * WM, CH = 32;
    constexpr int PL = PR + 1, PANEL = 4 * PL, RED = TG * WM * 256;                  // 16-byte units
    constexpr int PU = (4 * PR + NT - 1) / NT, PW = E == 1 ? 8 : 4, BE = BWD ? 1 : E, BW = BE == 1 ? 8 : 4;
    constexpr unsigned OOB = 0x80000000u;

    __shared__ __attribute__((aligned(16))) uint4 lds[PANEL > RED ? PANEL : RED];    // the panel, plane o = channels 8o..8o+7; at the end the groups' sums
    uint4 *panel = lds;
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

    // eight values from element `at` on, those of channel c and up (below Cred) at once or one by one; the others are zeros
    auto load8 = [&](__amdgpu_buffer_rsrc_t rs, auto e, bool ok, unsigned at, unsigned step, int c, uint32_t *v) __attribute__((always_inline)) {
        constexpr int N = decltype(e)::value;
        if constexpr (N == 8) {
            const float4 f = buffer_load4(rs, ok && c < Cred ? at * 2u : OOB);
            v[0] = __float_as_uint(f.x); v[1] = __float_as_uint(f.y); v[2] = __float_as_uint(f.z); v[3] = __float_as_uint(f.w);
        } else if constexpr (N == 2) {
#pragma unroll
            for (int j = 0; j < 4; j++) v[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(ok && c + 2 * j < Cred ? (at + 2 * j) * 2u : OOB), 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
                v[j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)(ok && c + j < Cred ? (at + j * step) * 2u : OOB), 0, 0);
        }
    };
    auto words = [&](const uint32_t *v, bool ones) __attribute__((always_inline)) {
        return ones ? make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16) : make_uint4(v[0], v[1], v[2], v[3]);
    };

    // ---- panel: thread -> (row, octet) pairs u = tid + i * NT
    const unsigned in_bytes = (unsigned)(p.g.N * Hi * Wi) * (unsigned)Cred * 2u;
    const __amdgpu_buffer_rsrc_t ars = owt_make_rsrc(p.a, in_bytes), mrs = owt_make_rsrc(MASKED ? p.mask : p.a, in_bytes);
    unsigned rowat[PU];
    bool rowok[PU];
#pragma unroll
    for (int i = 0; i < PU; i++) {
        const int row = (tid + i * NT) >> 2, pix = ps + row;
        rowok[i] = row < nrows && (unsigned)pix < (unsigned)(p.g.N * Hi * Wi);
        rowat[i] = (unsigned)pix * (unsigned)Cred;
    }
    uint32_t preg[PU][PW], yreg[MASKED ? PU : 1][PW];
    auto load_panel = [&](int ch) __attribute__((always_inline)) {
        const int c = ch * CH + (tid & 3) * 8;
#pragma unroll
        for (int i = 0; i < PU; i++) {
            load8(ars, std::integral_constant<int, E>(), rowok[i], rowat[i] + c, 1u, c, preg[i]);
            if (MASKED) load8(mrs, std::integral_constant<int, E>(), rowok[i], rowat[i] + c, 1u, c, yreg[MASKED ? i : 0]);
        }
    };
    auto store_panel = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PU; i++) {
            const int u = tid + i * NT, row = u >> 2;
            uint4 v = words(preg[i], E == 1);
            if (MASKED) v = mask_words16(v, words(yreg[MASKED ? i : 0], E == 1));
            if (row < PR) panel[(u & 3) * PL + row] = v;
        }
    };

    // ---- filters: this lane's column, two octets of a tap.  Forward: w[n][tap][c].  Backward-data: w[c][RS-1-tap][n].
    const __amdgpu_buffer_rsrc_t brs = owt_make_rsrc(p.b, (unsigned)p.Ncols * (unsigned)Cred * (unsigned)RS * 2u);
    const int n = n0 + li;
    uint32_t braw[2][2][BW];
    auto load_b = [&](int ch, int tap, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int c = ch * CH + 16 * k + 8 * lh;
            if (k == 1 && ch * CH + 16 >= Cred) {                             // (the same for every lane)
#pragma unroll
                for (int j = 0; j < BW; j++) braw[u][k][j] = 0u;
            } else if (BWD) {
                load8(brs, std::integral_constant<int, 1>(), n < p.Ncols, ((unsigned)c * RS + (RS - 1 - tap)) * (unsigned)p.Ncols + n, (unsigned)(RS * p.Ncols), c, braw[u][k]);
            } else {
                load8(brs, std::integral_constant<int, BE>(), n < p.Ncols, ((unsigned)n * RS + tap) * (unsigned)Cred + c, 1u, c, braw[u][k]);
            }
        }
    };

    typedef float acc16 __attribute__((ext_vector_type(16)));
    acc16 acc;
#pragma unroll
    for (int q = 0; q < 16; q++) acc[q] = 0.f;

    if (tid < 4) panel[tid * PL + PR] = make_uint4(0u, 0u, 0u, 0u);           // the row of zeros of every plane
    const int per_chunk = (RS - grp + TG - 1) / TG;                           // this group's taps: grp, grp + TG, ...
    const int nsteps = (ch_end - ch_beg) * per_chunk;
    int lch = ch_beg, ltap = grp;                                             // the step whose filters are loaded next
    auto load_next = [&](int u) __attribute__((always_inline)) {
        if (lch < ch_end) load_b(lch, ltap, u);
        ltap += TG;
        if (ltap >= RS) { ltap = grp; lch++; }
    };
    load_panel(ch_beg);
    load_next(0);
    load_next(1);
    int ch = ch_beg, tap = grp;
    for (int i = 0; i < nsteps; i += 2) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            if (i + u >= nsteps) break;
            if (tap == grp) {                                                 // a new chunk; every wavefront comes here once a chunk
                if (ch > ch_beg) __syncthreads();                             // everyone has its fragments of the old panel
                store_panel();
                __syncthreads();
                if (ch + 1 < ch_end) load_panel(ch + 1);
            }
            const int r = p.g.dS.div(tap), s = tap - r * S;
            const uint4 *arow = panel + lh * PL + (((inside >> tap) & 1u) ? prow + r * Wi + s : PR);
            bf16x8 a[2], f[2];
#pragma unroll
            for (int k = 0; k < 2; k++) {
                a[k] = __builtin_bit_cast(bf16x8, arow[2 * k * PL]);
                f[k] = __builtin_bit_cast(bf16x8, words(braw[u][k], BE == 1));
            }
            load_next(u);
#pragma unroll
            for (int k = 0; k < 2; k++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k], f[k], acc, 0, 0, 0);
            tap += TG;
            if (tap >= RS) { tap = grp; ch++; }
        }
    }

    // ---- the groups' sums, in the order of the groups; every wavefront adds up 16 / TG of the registers
    constexpr int QN = 16 / TG;
    const int q0 = grp * QN;
    float v[QN];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; q++) red[(grp * WM + wm) * 1024 + q * 64 + lane] = acc[q];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < QN; j++) {
        v[j] = red[wm * 1024 + (q0 + j) * 64 + lane];
#pragma unroll
        for (int g = 1; g < TG; g++) v[j] += red[(g * WM + wm) * 1024 + (q0 + j) * 64 + lane];
    }

    // ---- epilogue: register q of lane (li, lh) is pixel 8*(q/4) + 4*lh + q%4, column li.  Columns and pixels past the end get an offset
    // outside the descriptor: their stores are dropped.
    const bool part = p.splits > 1, relu = !BWD && !part && (p.flags & 2u), xm = BWD && !part && p.xmask != nullptr;
    const unsigned es = part ? 4u : 2u, out_bytes = (unsigned)p.M * (unsigned)p.Ncols * es;
    const __amdgpu_buffer_rsrc_t ors = owt_make_rsrc(part ? (const void *)(p.partial + (size_t)split * p.M * p.Ncols) : p.out, out_bytes);
    const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(xm ? p.xmask : p.a, xm ? out_bytes : 0u);
    const int mq = m0 + wm * 32 + 8 * (q0 / 4) + 4 * lh + q0 % 4;
    const float bias = (!BWD && !part && (p.flags & 1u) && n < p.Ncols) ? p.bias[n] : 0.f;
    const unsigned base = n < p.Ncols ? ((unsigned)mq * (unsigned)p.Ncols + (unsigned)n) * es : OOB;
    float x[QN];
    if (xm) {
#pragma unroll
        for (int j = 0; j < QN; j++)
            x[j] = bf16_to_f32((uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xrs, (int)(base + (unsigned)j * (unsigned)p.Ncols * 2u), 0, 0));
    }
#pragma unroll
    for (int j = 0; j < QN; j++) {
        float o = v[j] + bias;
        if (relu) o = o > 0.f ? o : 0.f;
        if (xm) o = x[j] > 0.f ? o : 0.f;
        const int at = (int)(base + (unsigned)j * (unsigned)p.Ncols * es);
        if (part) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ors, at, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(o), ors, at, 0, 0);
    }
}

}  // namespace owt
