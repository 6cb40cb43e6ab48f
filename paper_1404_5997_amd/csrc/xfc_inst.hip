// Instantiations of the fully-connected shard's kernels on the bf16 matrix unit.
#include <type_traits>

#include "xfc.hpp"
#include "owt_host.hpp"

namespace owt {

template <bool BF>
static hipError_t fwd(const GemmParams &p, hipStream_t s)
{
    typedef EpiFwd<typename std::conditional<BF, bf16_t, float>::type> Epi;
    hipLaunchKernelGGL((xfc_fwd_kernel<Epi, BF>), dim3(p.tiles_m * p.tiles_n, p.splits), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<Epi>(p, s);
    return e;
}

template <bool BF>
static hipError_t bwd(const GemmParams &pd, const GemmParams &pf, hipStream_t s)
{
    const int wgs = pd.tiles_m * pd.tiles_n + pf.tiles_m * pf.tiles_n;
    if (pf.mask) hipLaunchKernelGGL((xfc_bwd_kernel<BF, true>), dim3(wgs), dim3(256), 0, s, pd, pf);
    else hipLaunchKernelGGL((xfc_bwd_kernel<BF, false>), dim3(wgs), dim3(256), 0, s, pd, pf);
    return hipGetLastError();
}

hipError_t owt_launch_xfc_fwd(bool bf16, const GemmParams &p, hipStream_t s) { return bf16 ? fwd<true>(p, s) : fwd<false>(p, s); }

hipError_t owt_launch_xfc_bwd(bool bf16, const GemmParams *pd, const GemmParams *pf, hipStream_t s)
{
    // a product that is not wanted has no tiles; the kernel takes N, O and I from the filter product's frame
    GemmParams d, f;
    if (pf) f = *pf;
    else { f = *pd; f.M = pd->Kd; f.Kd = pd->M; f.Ncols = pd->Ncols; f.tiles_m = 0; f.dbias = nullptr; }
    if (pd) d = *pd;
    else { d = *pf; d.tiles_m = 0; }
    if (pd && pf && (pd->M != pf->Kd || pd->Kd != pf->M || pd->Ncols != pf->Ncols || pd->mask != pf->mask)) return hipErrorInvalidValue;
    return bf16 ? bwd<true>(d, f, s) : bwd<false>(d, f, s);
}

}  // namespace owt
