// Instantiations of the bf16 stride-1 kernel for layers of few tiles, for one pass.
// Built twice: -DOWT_INST_PASS={0,1}.
#include "dconv16s.hpp"
#include "owt_host.hpp"

#ifndef OWT_INST_PASS
#error "define OWT_INST_PASS (0 fwd, 1 bwd-data)"
#endif

namespace owt {

constexpr bool kBwd = OWT_INST_PASS == 1;
typedef std::conditional<kBwd, EpiData<bf16_t>, EpiFwd<bf16_t>>::type OE;

template <int V, int PR, int E>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr DConv16SVariant v = kDConv16SVariants[V];
    const dim3 grid(p.tiles_m * p.tiles_n, p.splits), block(64 * v.WM * v.TG);
#if OWT_INST_PASS == 1
    if (p.mask) {
        if constexpr (E > 1 || dconv16s_masked_fits(v, PR)) hipLaunchKernelGGL((dconv16s_kernel<kBwd, v.WM, v.TG, PR, E, true>), grid, block, 0, s, p);
        else return hipErrorInvalidValue;
    } else
#endif
    hipLaunchKernelGGL((dconv16s_kernel<kBwd, v.WM, v.TG, PR, E, false>), grid, block, 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<OE>(p, s);
    return e;
}

template <int V>
static hipError_t size(int pr, const GemmParams &p, hipStream_t s)
{
    constexpr DConv16SVariant v = kDConv16SVariants[V];
    if (p.g.R * p.g.S < v.TG || p.g.R * p.g.S > 32) return hipErrorInvalidValue;
    const int e = p.Cred % 8 == 0 ? 8 : p.Cred % 2 == 0 ? 2 : 1;
    if (pr <= v.prs[0]) return e == 8 ? go<V, v.prs[0], 8>(p, s) : e == 2 ? go<V, v.prs[0], 2>(p, s) : go<V, v.prs[0], 1>(p, s);
    if (pr <= v.prs[1]) return e == 8 ? go<V, v.prs[1], 8>(p, s) : e == 2 ? go<V, v.prs[1], 2>(p, s) : go<V, v.prs[1], 1>(p, s);
    if (pr <= v.prs[2]) return e == 8 ? go<V, v.prs[2], 8>(p, s) : e == 2 ? go<V, v.prs[2], 2>(p, s) : go<V, v.prs[2], 1>(p, s);
    return hipErrorInvalidValue;
}

#if OWT_INST_PASS == 0
hipError_t owt_launch_dconv16s_fwd(int variant, int pr, const GemmParams &p, hipStream_t s)
#else
hipError_t owt_launch_dconv16s_data(int variant, int pr, const GemmParams &p, hipStream_t s)
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
