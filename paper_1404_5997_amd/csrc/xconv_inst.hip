// Instantiations of the split-operand stride-1 kernel for one pass and one way of loading the panel.
// Built five times: -DOWT_INST_PASS={0,1} -DOWT_INST_VEC={0,1}, and {0} {2} (strided forward as blocks).
#include "xconv.hpp"
#include "owt_host.hpp"

#if !defined(OWT_INST_PASS) || !defined(OWT_INST_VEC)
#error "define OWT_INST_PASS (0 fwd, 1 bwd-data) and OWT_INST_VEC (XC_SCALAR, XC_VEC, XC_BLOCKS)"
#endif

namespace owt {

#if OWT_INST_PASS == 0
typedef EpiFwd<float> OE;
constexpr bool kBwd = false;
#define OWT_XFN_(v) owt_launch_xconv_fwd_vec##v
#else
typedef EpiData<float> OE;
constexpr bool kBwd = true;
#define OWT_XFN_(v) owt_launch_xconv_data_vec##v
#endif
#define OWT_XFN(v) OWT_XFN_(v)

template <int WM, int WN, int MB, int PR, int OCC>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    const dim3 grid(p.tiles_m * p.tiles_n, p.splits), block(64 * WM * WN);
    if constexpr (kBwd) {
        if (p.mask) {
            hipLaunchKernelGGL((xconv_kernel<OE, kBwd, WM, WN, MB, PR, OCC, OWT_INST_VEC, true>), grid, block, 0, s, p);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((xconv_kernel<OE, kBwd, WM, WN, MB, PR, OCC, OWT_INST_VEC, false>), grid, block, 0, s, p);
    return hipGetLastError();
}

#if OWT_INST_VEC == 2
hipError_t owt_launch_xconv_fwd_blocks(int variant, int pr, const GemmParams &p0, void *ws, hipStream_t s)
#else
hipError_t OWT_XFN(OWT_INST_VEC)(int variant, int pr, const GemmParams &p0, void *ws, hipStream_t s)
#endif
{
    GemmParams p = p0;
    const Geom &g = p0.g;
    const int nblocks = p0.tiles_n * 2 * kXConvVariants[variant].WN;
#if OWT_INST_VEC == 2
    p.g.R = (g.R + g.sh - 1) / g.sh;                     // the kernel's taps are blocks
    p.g.S = (g.S + g.sw - 1) / g.sw;
    p.R0 = g.R; p.S0 = g.S;
#endif
    p.b0 = p0.b;
    const int RS = p.g.R * p.g.S;
    const long threads = (long)p0.ksteps * RS * nblocks * 64;
    const unsigned blocks = (unsigned)((threads + 255) / 256 > 8192 ? 8192 : (threads + 255) / 256);
#if OWT_INST_VEC == 2
    hipLaunchKernelGGL(xconv_pack_blocks_kernel, dim3(blocks), dim3(256), 0, s, (const float *)p0.b, (uint4 *)ws, g, p.g.R, p.g.S,
                       p0.ksteps, nblocks);
#else
    hipLaunchKernelGGL((xconv_pack_kernel<kBwd>), dim3(blocks), dim3(256), 0, s, (const float *)p0.b, (uint4 *)ws, g.K, RS, g.C,
                       p0.ksteps, nblocks);
#endif
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.b = ws;
    e = hipErrorInvalidValue;
    if (variant == 0) {
        if (pr <= 160) e = go<2, 2, 2, 160, 2>(p, s);
        else if (pr <= 288) e = go<2, 2, 2, 288, 2>(p, s);
    } else if (variant == 1) {
        if (pr <= 288) e = go<4, 1, 2, 288, 2>(p, s);
        else if (pr <= 384) e = go<4, 1, 2, 384, 2>(p, s);
        else if (pr <= 512) e = go<4, 1, 2, 512, 2>(p, s);
    } else if (variant == 2) {
        if (pr <= 160) e = go<2, 1, 2, 160, 2>(p, s);
        else if (pr <= 288) e = go<2, 1, 2, 288, 2>(p, s);
    } else if (variant == 3) {
        if (pr <= 160) e = go<4, 1, 1, 160, 3>(p, s);
        else if (pr <= 288) e = go<4, 1, 1, 288, 3>(p, s);
    }
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<OE>(p, s);
    return e;
}

}  // namespace owt
