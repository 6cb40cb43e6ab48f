// Instantiations of the split-operand stride-1 filter-gradient kernel.
#include "xfilter.hpp"
#include "owt_host.hpp"

namespace owt {

template <int V>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr XFilterVariant v = kXFilterVariants[V];
    const int tiles = p.tiles_m * p.tiles_n;
    const dim3 grid(v.TG > 1 ? owt_split_major_grid(tiles, p.splits) : owt_split_major_wave_grid(tiles, p.splits));
    if (p.mask) hipLaunchKernelGGL((xfilter_kernel<v.KB, v.S, v.TG, true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((xfilter_kernel<v.KB, v.S, v.TG, false>), grid, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFilter>(p, s);
    return e;
}

hipError_t owt_launch_xfilter(int variant, const GemmParams &p, hipStream_t s)
{
    if (p.g.S != kXFilterVariants[variant].S) return hipErrorInvalidValue;
    switch (variant) {
    case 0: return go<0>(p, s);
    case 1: return go<1>(p, s);
    case 2: return go<2>(p, s);
    case 3: return go<3>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace owt
