// Instantiations of the split-operand filter-gradient kernel for any geometry.
#include "xgather.hpp"
#include "owt_host.hpp"

namespace owt {

template <int V>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr XGatherVariant v = kXGatherVariants[V];
    const dim3 grid(owt_split_major_grid(p.tiles_m * p.tiles_n, p.splits));
    if (p.mask) hipLaunchKernelGGL((xgather_kernel<v.KB, v.CB, v.TG, true>), grid, dim3(64 * v.TG), 0, s, p);
    else hipLaunchKernelGGL((xgather_kernel<v.KB, v.CB, v.TG, false>), grid, dim3(64 * v.TG), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFilter>(p, s);
    return e;
}

hipError_t owt_launch_xgather(int variant, const GemmParams &p, hipStream_t s)
{
    switch (variant) {
    case 0: return go<0>(p, s);
    case 1: return go<1>(p, s);
    case 2: return go<2>(p, s);
    case 3: return go<3>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace owt
