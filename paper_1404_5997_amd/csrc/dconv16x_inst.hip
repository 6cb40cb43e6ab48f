// Instantiations of the pipelined bf16-MFMA kernel for any channel counts, and for strided forward passes over blocks of pixels.
// Built three times: -DOWT_INST_PASS={0,1,2} (forward, backward-data, strided forward).
#include "dconv_bf16p.hpp"
#include "owt_host.hpp"

#ifndef OWT_INST_PASS
#error "define OWT_INST_PASS (0 fwd, 1 bwd-data, 2 strided forward over blocks)"
#endif

namespace owt {

constexpr bool kBwd = OWT_INST_PASS == 1, kBlocks = OWT_INST_PASS == 2;
typedef std::conditional<kBwd, EpiData<bf16_t>, EpiFwd<bf16_t>>::type OE;

template <int PR, int LOAD, bool MASKED>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr int OCC = LOAD == DP_EVEN && !MASKED ? 3 : 2;
    hipLaunchKernelGGL((dconv16p_kernel<OE, kBwd, PR, 2, OCC, LOAD, MASKED>), dim3(p.tiles_m * p.tiles_n, p.splits), dim3(256), 0, s, p);
    return hipGetLastError();
}

template <int PR>
static hipError_t load(const GemmParams &p, hipStream_t s)
{
#if OWT_INST_PASS == 2
    return go<PR, DP_BLOCKS, false>(p, s);
#else
#if OWT_INST_PASS == 1
    if (p.mask) return p.Cred % 2 ? go<PR, DP_ODD, true>(p, s) : go<PR, DP_EVEN, true>(p, s);
#endif
    return p.Cred % 2 ? go<PR, DP_ODD, false>(p, s) : go<PR, DP_EVEN, false>(p, s);
#endif
}

#if OWT_INST_PASS == 0
hipError_t owt_launch_dconv16x_fwd(int pr, const GemmParams &p0, void *ws, hipStream_t s)
#elif OWT_INST_PASS == 1
hipError_t owt_launch_dconv16x_data(int pr, const GemmParams &p0, void *ws, hipStream_t s)
#else
hipError_t owt_launch_dconv16x_blocks(int pr, const GemmParams &p0, void *ws, hipStream_t s)
#endif
{
    GemmParams p = p0;
    const Geom &g = p0.g;
    if (kBlocks) {                                       // the kernel's taps are blocks
        p.g.R = (g.R + g.sh - 1) / g.sh;
        p.g.S = (g.S + g.sw - 1) / g.sw;
        p.R0 = g.R; p.S0 = g.S;
        p.b0 = p0.b;
    }
    if (p.g.R * p.g.S < 2 || p.g.R * p.g.S > 32 || (kBlocks && p.ksteps > 8)) return hipErrorInvalidValue;
    const long threads = (long)p.Ncols * p.g.R * p.g.S * p.ksteps * 4;
    hipLaunchKernelGGL((dconv16x_pack_kernel<kBwd, kBlocks>), dim3((unsigned)((threads + 255) / 256 > 8192 ? 8192 : (threads + 255) / 256)), dim3(256), 0, s,
                       (const uint16_t *)p0.b, (uint4 *)ws, g, p.g.R, p.g.S, p.ksteps * 4);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.b = ws;
    if (pr <= 288) e = load<288>(p, s);
    else if (pr <= 384) e = load<384>(p, s);
    else if (pr <= 512) e = load<512>(p, s);
    else return hipErrorInvalidValue;
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<OE>(p, s);
    return e;
}

}  // namespace owt
