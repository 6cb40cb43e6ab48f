// Instantiations of the bf16 filter-gradient kernels with the reduction over images (stride 1, and any geometry).
// Built twice: -DOWT_INST_MASKED={0,1}.
#include "igather16.hpp"
#include "owt_host.hpp"

#ifndef OWT_INST_MASKED
#error "define OWT_INST_MASKED (1: the call masks dz itself)"
#endif

namespace owt {

template <int V, bool ZP, bool XP>
static hipError_t go(const GemmParams &p, hipStream_t s)
{
    constexpr IFilter16Variant v = kIFilter16Variants[V];
    const dim3 grid(owt_split_major_grid(p.tiles_m * p.tiles_n, p.splits));
    hipLaunchKernelGGL((ifilter16_kernel<v.KB, v.CB, v.S, ZP, XP, OWT_INST_MASKED != 0>), grid, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFilter>(p, s);
    return e;
}

// filters / channels in pairs where a tile has two blocks of them and their number is even
template <int V>
static hipError_t pairs(const GemmParams &p, hipStream_t s)
{
    constexpr IFilter16Variant v = kIFilter16Variants[V];
    const bool zp = v.KB == 2 && p.g.K % 2 == 0, xp = v.CB == 2 && p.g.C % 2 == 0;
    if constexpr (v.KB == 2 && v.CB == 2) { if (zp && xp) return go<V, true, true>(p, s); }
    if constexpr (v.KB == 2) { if (zp) return go<V, true, false>(p, s); }
    if constexpr (v.CB == 2) { if (xp) return go<V, false, true>(p, s); }
    return go<V, false, false>(p, s);
}

#if OWT_INST_MASKED
hipError_t owt_launch_ifilter16_masked(int variant, const GemmParams &p, hipStream_t s)
#else
hipError_t owt_launch_ifilter16(int variant, const GemmParams &p, hipStream_t s)
#endif
{
    if (variant < 0 || variant >= kNumIFilter16Variants || p.g.S != kIFilter16Variants[variant].S) return hipErrorInvalidValue;
    switch (variant) {
    case 0: return pairs<0>(p, s);
    case 1: return pairs<1>(p, s);
    case 2: return pairs<2>(p, s);
    case 3: return pairs<3>(p, s);
    case 4: return pairs<4>(p, s);
    case 5: return pairs<5>(p, s);
    case 6: return pairs<6>(p, s);
    default: return hipErrorInvalidValue;
    }
}

template <int V, bool ZP>
static hipError_t go_any(const GemmParams &p, hipStream_t s)
{
    constexpr IGather16Variant v = kIGather16Variants[V];
    hipLaunchKernelGGL((igather16_kernel<v.KB, v.CB, ZP, OWT_INST_MASKED != 0>), dim3(owt_split_major_grid(p.tiles_m * p.tiles_n, p.splits)), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFilter>(p, s);
    return e;
}

#if OWT_INST_MASKED
hipError_t owt_launch_igather16_masked(int variant, const GemmParams &p, hipStream_t s)
#else
hipError_t owt_launch_igather16(int variant, const GemmParams &p, hipStream_t s)
#endif
{
    switch (variant) {
    case 0: return go_any<0, false>(p, s);
    case 1: return p.g.K % 2 ? go_any<1, false>(p, s) : go_any<1, true>(p, s);
    case 2: return go_any<2, false>(p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace owt
