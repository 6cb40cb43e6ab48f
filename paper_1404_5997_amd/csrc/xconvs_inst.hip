// Instantiations of the split-operand stride-1 kernel for layers of few tiles, for one pass.
// Built twice: -DOWT_INST_PASS={0,1}.
#include "xconvs.hpp"
#include "owt_host.hpp"

#ifndef OWT_INST_PASS
#error "define OWT_INST_PASS (0 fwd, 1 bwd-data)"
#endif

namespace owt {

constexpr bool kBwd = OWT_INST_PASS == 1;
typedef std::conditional<kBwd, EpiData<float>, EpiFwd<float>>::type OE;

template <int V, int PR, bool VEC>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr XConvSVariant v = kXConvSVariants[V];
    const dim3 grid(p.tiles_m * p.tiles_n, p.splits), block(64 * v.WM * v.TG);
#if OWT_INST_PASS == 1
    if (p.mask) hipLaunchKernelGGL((xconvs_kernel<kBwd, v.WM, v.TG, PR, VEC, true>), grid, block, 0, s, p);
    else
#endif
    hipLaunchKernelGGL((xconvs_kernel<kBwd, v.WM, v.TG, PR, VEC, false>), grid, block, 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<OE>(p, s);
    return e;
}

template <int V>
static hipError_t size(int pr, const GemmParams &p, hipStream_t s)
{
    constexpr XConvSVariant v = kXConvSVariants[V];
    if (p.g.R * p.g.S < v.TG || p.g.R * p.g.S > 32) return hipErrorInvalidValue;
    const bool vec = p.Cred % 4 == 0;
    if (pr <= v.prs[0]) return vec ? go<V, v.prs[0], true>(p, s) : go<V, v.prs[0], false>(p, s);
    if (pr <= v.prs[1]) return vec ? go<V, v.prs[1], true>(p, s) : go<V, v.prs[1], false>(p, s);
    if (pr <= v.prs[2]) return vec ? go<V, v.prs[2], true>(p, s) : go<V, v.prs[2], false>(p, s);
    return hipErrorInvalidValue;
}

#if OWT_INST_PASS == 0
hipError_t owt_launch_xconvs_fwd(int variant, int pr, const GemmParams &p, hipStream_t s)
#else
hipError_t owt_launch_xconvs_data(int variant, int pr, const GemmParams &p, hipStream_t s)
#endif
{
    switch (variant) {
    case 0: return size<0>(pr, p, s);
    case 1: return size<1>(pr, p, s);
    case 2: return size<2>(pr, p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace owt
