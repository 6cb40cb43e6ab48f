// Filter gradient of any convolution, fp32 storage, on the bf16 matrix unit with operands split in three (split3.hpp).
//
//   dw[k][j] = sum over (p,q), images n of  dz[n,p,q,k] * x[n, p*sh + r - pad_h, q*sw + s - pad_w, c],   j = (r*S + s)*C + c
//
// (Section 4 of the paper, backward step 2.)  As in xfilter.hpp a matrix instruction takes 16 images at one output
// position, operands are loaded 4 bytes per lane for eight images, split in registers, and there is no LDS and no
// barrier.  Here the columns are the filter's (r, s, c) places packed densely, whatever they are: a lane keeps its
// place's byte offset and (r, s), so any stride and any channel count will do -- the first layer's 11 x 11 x 3 = 363
// places fill 11.3 of 12 blocks -- but neighbouring positions share no fragments.  A wavefront holds KB x CB blocks and
// splits KB + CB fragments per position for 6 * KB * CB matrix instructions: at 2 x 3 the vector instructions take longer
// than the matrix instructions they are issued between.
//
// Loads run two positions ahead (one was 3 us slower, and 2 x 4 blocks with one 4 us).  Where four wavefronts share a tile (TG = 4,
// as in xfilter.hpp), one position ahead, which leaves room for two wavefronts a SIMD: 8 images 32x32x3 -> 16, 5x5, masked 14.2 -> 10.9
// us, 32x64 tiles; 3 images 224x224x3 -> 48, 11x11 stride 4 40 -> 31.  Long walks stay with 2 x 3 blocks (below: 154 us against 169).
//
// Measured, first layer (128 images, 224x224x3 -> 64, 11x11 stride 4) with the reduce pass: 159 us on the fp32 instruction,
// 144 here (125 TFLOP/s); four wavefronts to a work-group, which helps xfilter.hpp by 2 %, cost small layers 2 us and won
// nothing.  8 images 32x32x3 -> 16, 5x5 (gather kernel before): 20.7 -> 15.3 us, half of it the reduce pass's launch.
#pragma once
#include <type_traits>

#include "xfilter.hpp"

namespace owt {

template <int KB, int CB, int TG, bool MASKED>
__global__ void __launch_bounds__(64 * TG, TG > 1 ? 2 : 1) xgather_kernel(const GemmParams p)
{
    constexpr int M = 6 * KB * CB, F = KB + CB;    // matrix instructions and fragments per position
    constexpr int SETS = TG > 1 ? 1 : 2;           // positions whose loads are in flight; two wavefronts a SIMD have registers for one

    const Geom &g = p.g;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5, wave = TG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    int tile, split;
    if (!owt_split_major_wg(p.tiles_m * p.tiles_n, p.splits, tile, split)) return;
    const int kt = tile / p.tiles_n, ct = tile - kt * p.tiles_n;
    const int k0 = kt * 32 * KB, j0 = ct * 32 * CB;

    const int P = g.P, Q = g.Q, total = ((g.N + 15) >> 4) * P * Q;
    // the work-group's positions, and this wavefront's part of them
    const int g_beg = min(total, split * p.ksteps_per_split), g_end = min(total, g_beg + p.ksteps_per_split), sub = (p.ksteps_per_split + TG - 1) / TG;
    const int o_beg = min(g_end, g_beg + wave * sub), o_end = min(g_end, o_beg + sub);

    const unsigned imgx = (unsigned)(g.H * g.W * g.C) * 4u, imgz = (unsigned)(P * Q * g.K) * 4u;
    // what must read as zero gets an offset of xall or zall, the end of its tensor; with the scalar part added it stays below
    // 2^32 (host-checked)
    const unsigned xall = imgx * (unsigned)g.N, zall = imgz * (unsigned)g.N;
    const __amdgpu_buffer_rsrc_t xrs = owt_make_rsrc(p.b, xall), zrs = owt_make_rsrc(p.a, zall);
    const __amdgpu_buffer_rsrc_t yrs = owt_make_rsrc(MASKED ? p.mask : p.a, zall);

    // This lane's places: byte offset from the window's corner (of the image 8*lh past the group's first), filter row and
    // column.  A place past the last is far outside every image.  Images past the last and filters past a ragged tile:
    // as in xfilter.hpp.
    int coff[CB], cr[CB], cs[CB];
#pragma unroll
    for (int cb = 0; cb < CB; cb++) {
        const int j = j0 + cb * 32 + li, rs = g.dC.div(j), r = g.dS.div(rs);
        cr[cb] = j < p.Ncols ? r : 0x10000000;
        cs[cb] = rs - r * g.S;
        coff[cb] = ((r * g.W + cs[cb]) * g.C + (j - rs * g.C)) * 4 + (int)((unsigned)(8 * lh) * imgx);
    }
    const unsigned zo = (unsigned)(8 * lh) * imgz + (unsigned)(k0 + li) * 4u;

    split_acc big[KB][CB], small[KB][CB];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int cb = 0; cb < CB; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) big[kb][cb][e] = small[kb][cb][e] = 0.f;
    };
    float db[KB];
#pragma unroll
    for (int kb = 0; kb < KB; kb++) db[kb] = 0.f;

    float sx = 1.f, sz = 1.f;                       // scales of x and dz in a careful run
    auto walk = [&](auto db_tag, auto careful_tag) __attribute__((always_inline)) {
        constexpr bool DB = decltype(db_tag)::value, CAREFUL = decltype(careful_tag)::value;
        if (o_beg >= o_end) return;
        int o = o_beg, n0, pp, qq;
        {
            const int grp = o_beg / (P * Q), rem = o_beg - grp * (P * Q);
            n0 = 16 * grp; pp = rem / Q; qq = rem - pp * Q;
        }
        // the position that loads are issued for: scalar offsets of its window corner and its dz row, per-lane offsets of
        // its places (outside the descriptor where the place is outside the image, or the walk is over)
        unsigned xoff = 0u, zoff = 0u;
        unsigned place[CB];
        int zbase = 0;
        auto aim = [&]() __attribute__((always_inline)) {
            const int h0 = pp * g.sh - g.ph, w0 = qq * g.sw - g.pw;
            const bool live = o < o_end;
            // the corner may lie outside the image: its offset is folded into the lanes' part, modulo 2^32
            xoff = live ? (unsigned)n0 * imgx : 0u;
            const int corner = (h0 * g.W + w0) * g.C * 4;
#pragma unroll
            for (int cb = 0; cb < CB; cb++) {
                const bool in = (unsigned)(h0 + cr[cb]) < (unsigned)g.H && (unsigned)(w0 + cs[cb]) < (unsigned)g.W;
                place[cb] = live && in ? (unsigned)(coff[cb] + corner) : xall;
            }
            zoff = live ? (unsigned)n0 * imgz + (unsigned)((pp * Q + qq) * g.K) * 4u : 0u;
            zbase = (int)(live ? zo : zall);
            o++;
            const bool row_end = qq + 1 == Q, image_end = row_end && pp + 1 == P;
            qq = row_end ? 0 : qq + 1;
            pp = image_end ? 0 : (row_end ? pp + 1 : pp);
            n0 = image_end ? n0 + 16 : n0;
        };
        float xr[SETS][CB][8], zr[SETS][KB][8], yr[SETS][MASKED ? KB : 1][8];
        auto load = [&](int set, int f) __attribute__((always_inline)) {
            if (f < CB) {
#pragma unroll
                for (int e = 0; e < 8; e++)
                    xr[set][f < CB ? f : 0][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrs, (int)place[f < CB ? f : 0], (int)(xoff + (unsigned)e * imgx), 0));
            } else {
                const int kb = f - CB;
#pragma unroll
                for (int e = 0; e < 8; e++)
                    zr[set][kb][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zrs, zbase + kb * 128, (int)(zoff + (unsigned)e * imgz), 0));
                if (MASKED) {
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        yr[set][MASKED ? kb : 0][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(yrs, zbase + kb * 128, (int)(zoff + (unsigned)e * imgz), 0));
                }
            }
        };
        auto split = [&](float (&v)[8], float scale, split_frag (&f)[3]) __attribute__((always_inline)) {
            if constexpr (CAREFUL) {
                float u[8];
#pragma unroll
                for (int e = 0; e < 8; e++) u[e] = v[e] * scale;
                split3_careful(u, f);
            } else {
                split3_plain(v, f);
            }
        };
        float run_db[KB];                            // the bias gradient's sum of 16 positions: one long chain of additions rounds more
#pragma unroll
        for (int kb = 0; kb < KB; kb++) run_db[kb] = 0.f;
        auto split_f = [&](int set, int f, split_frag (&fz)[KB][3], split_frag (&fx)[CB][3]) __attribute__((always_inline)) {
            if (f < CB) {
                split(xr[set][f < CB ? f : 0], sx, fx[f < CB ? f : 0]);
            } else {
                const int kb = f - CB;
                float (&z)[8] = zr[set][kb];
                if (MASKED) {
#pragma unroll
                    for (int e = 0; e < 8; e++) z[e] = yr[set][MASKED ? kb : 0][e] > 0.f ? z[e] : 0.f;
                }
                if (DB) run_db[kb] += ((z[0] + z[1]) + (z[2] + z[3])) + ((z[4] + z[5]) + (z[6] + z[7]));
                split(z, sz, fz[kb]);
            }
        };

        split_frag az[KB][3], bx[CB][3];
        aim();
#pragma unroll
        for (int set = 0; set < SETS; set++) {
#pragma unroll
            for (int f = 0; f < F; f++) load(set, f);
            aim();
        }
#pragma unroll
        for (int f = 0; f < F; f++) { split_f(0, f, az, bx); load(0, f); }
        aim();
        // (past the walk's end a position's operands are zeros: the second of the last pair may be one)
        for (int i = o_beg; i < o_end; i += SETS) {
#pragma unroll
            for (int u = 0; u < SETS; u++) {
                // the products of position i + u, one phase per fragment of position i + u + 1: its vector instructions are
                // spread between the phase's matrix instructions, then its raw registers are loaded for position i + u + 1 + SETS
                split_frag nz[KB][3], nx[CB][3];
#pragma unroll
                for (int f = 0; f < F; f++) {
                    split_f((u + 1) % SETS, f, nz, nx);
                    load((u + 1) % SETS, f);
                    constexpr int PH = M / F;
#pragma unroll
                    for (int q = f * PH; q < (f == F - 1 ? M : (f + 1) * PH); q++) {
                        constexpr int PA[6] = {0, 2, 0, 1, 1, 0}, PB[6] = {0, 0, 2, 1, 0, 1};
                        const int kb = q / (6 * CB), e = q / CB % 6, cb = q % CB;
                        split_acc &acc = e == 0 ? big[kb][cb] : small[kb][cb];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(az[kb][PA[e]], bx[cb][PB[e]], acc, 0, 0, 0);
                    }
                    constexpr int VPM = (44 + (MASKED ? 16 : 0) + (DB ? 8 : 0) + PH - 1) / PH;
#pragma unroll
                    for (int q = 0; q < PH; q++) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // a matrix instruction
                        __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);     // vector instructions in its shadow
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                aim();
#pragma unroll
                for (int kb = 0; kb < KB; kb++)
#pragma unroll
                    for (int e = 0; e < 3; e++) az[kb][e] = nz[kb][e];
#pragma unroll
                for (int cb = 0; cb < CB; cb++)
#pragma unroll
                    for (int e = 0; e < 3; e++) bx[cb][e] = nx[cb][e];
            }
            if (DB && (((i - o_beg) & (16 - SETS)) == 16 - SETS || i + SETS >= o_end)) {
#pragma unroll
                for (int kb = 0; kb < KB; kb++) { db[kb] += run_db[kb]; run_db[kb] = 0.f; }
            }
        }
    };

    clear();
    const bool do_db = ct == 0 && p.dbias != nullptr;
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
            for (int cb = 0; cb < CB; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const float v = big[kb][cb][e] + small[kb][cb][e];
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

    // register e of lane (li, lh): filter 8*(e/4) + 4*lh + e%4 of its block, place li
    const bool part = p.splits > 1;
    float *out = part ? p.partial + (size_t)split * p.M * p.Ncols : (float *)p.out;
    auto store = [&](int kb, int cb, int e, float v) __attribute__((always_inline)) {
        const int j = j0 + cb * 32 + li, k = k0 + kb * 32 + 8 * (e / 4) + 4 * lh + e % 4;
        if (j >= p.Ncols || k >= g.K) return;
        const size_t at = (size_t)k * p.Ncols + j;
        if (part) out[at] = v;
        else out[at] = p.alpha * v + (p.beta != 0.f ? p.beta * out[at] : 0.f);
    };
    auto store_db = [&](int kb, float v) __attribute__((always_inline)) {
        const int k = k0 + kb * 32 + li;
        if (lh || k >= g.K) return;
        if (part) p.dbias_partial[(size_t)split * p.M + k] = v;
        else p.dbias[k] = p.alpha * v + (p.beta != 0.f ? p.beta * p.dbias[k] : 0.f);
    };
    if constexpr (TG == 1) {
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int e = 0; e < 16; e++) store(kb, cb, e, (big[kb][cb][e] + small[kb][cb][e]) * unscale);
        if (do_db) {
#pragma unroll
            for (int kb = 0; kb < KB; kb++) store_db(kb, db[kb] + __shfl_xor(db[kb], 32));
        }
    } else {
        // the wavefronts' sums, added in pairs
        constexpr int V = KB * CB * 16;
        __shared__ float red[TG * (V + KB) * 64];
        float *mine = red + wave * (V + KB) * 64 + lane;
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int e = 0; e < 16; e++) mine[((kb * CB + cb) * 16 + e) * 64] = (big[kb][cb][e] + small[kb][cb][e]) * unscale;
#pragma unroll
        for (int kb = 0; kb < KB; kb++) mine[(V + kb) * 64] = db[kb] + __shfl_xor(db[kb], 32);
        __syncthreads();
        static_assert(TG == 4, "four wavefronts' sums in two pairs");
        for (int v = wave; v < V + KB; v += TG) {
            const float *at = red + v * 64 + lane;
            const float sum = (at[0] + at[(V + KB) * 64]) + (at[2 * (V + KB) * 64] + at[3 * (V + KB) * 64]);
            if (v < V) store(v / (CB * 16), v / 16 % CB, v % 16, sum);
            else if (do_db) store_db(v - V, sum);
        }
    }
}

}  // namespace owt
