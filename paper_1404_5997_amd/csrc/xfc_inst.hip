// Instantiations of the fully-connected shard's kernels on the bf16 matrix unit.
#include "xfc.hpp"
#include "xfc16.hpp"
#include "xfcs.hpp"
#include "owt_host.hpp"

namespace owt {

static hipError_t fwd32(const GemmParams &p, hipStream_t s)
{
    hipLaunchKernelGGL((xfc_fwd_kernel<EpiFwd<float>>), dim3(p.tiles_m * p.tiles_n, p.splits), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFwd<float>>(p, s);
    return e;
}

static hipError_t fwd16(const GemmParams &p, hipStream_t s)
{
    const dim3 grid(p.tiles_m * p.tiles_n, p.splits);
    if (p.Kd % 2 == 0) hipLaunchKernelGGL((xfc16_fwd_kernel<true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((xfc16_fwd_kernel<false>), grid, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && p.splits > 1) e = launch_splitk_reduce<EpiFwd<bf16_t>>(p, s);
    return e;
}

static hipError_t bwd32(const GemmParams &pd, const GemmParams &pf, int wgs, hipStream_t s)
{
    if (pf.mask) hipLaunchKernelGGL((xfc_bwd_kernel<true>), dim3(wgs), dim3(256), 0, s, pd, pf);
    else hipLaunchKernelGGL((xfc_bwd_kernel<false>), dim3(wgs), dim3(256), 0, s, pd, pf);
    return hipGetLastError();
}

template <bool OE, bool IE>
static hipError_t bwd16(const GemmParams &pd, const GemmParams &pf, int wgs, hipStream_t s)
{
    if (pf.mask) hipLaunchKernelGGL((xfc16_bwd_kernel<true, OE, IE>), dim3(wgs), dim3(256), 0, s, pd, pf);
    else hipLaunchKernelGGL((xfc16_bwd_kernel<false, OE, IE>), dim3(wgs), dim3(256), 0, s, pd, pf);
    return hipGetLastError();
}

hipError_t owt_launch_xfcs_fwd(bool bf16, const GemmParams &p, hipStream_t s)
{
    const dim3 grid(p.tiles_m * p.tiles_n);
    if (!bf16) hipLaunchKernelGGL((xfcs_fwd_kernel<float, false>), grid, dim3(1024), 0, s, p);
    else if (p.Kd % 2) hipLaunchKernelGGL((xfcs_fwd_kernel<bf16_t, true>), grid, dim3(1024), 0, s, p);
    else hipLaunchKernelGGL((xfcs_fwd_kernel<bf16_t, false>), grid, dim3(1024), 0, s, p);
    return hipGetLastError();
}

hipError_t owt_launch_xfc_fwd(bool bf16, const GemmParams &p, hipStream_t s) { return bf16 ? fwd16(p, s) : fwd32(p, s); }

hipError_t owt_launch_xfc_bwd(bool bf16, const GemmParams *pd, const GemmParams *pf, hipStream_t s)
{
    // a product that is not wanted has no tiles; the kernel takes N, O and I from the filter product's frame
    GemmParams d, f;
    if (pf) f = *pf;
    else { f = *pd; f.M = pd->Kd; f.Kd = pd->M; f.Ncols = pd->Ncols; f.tiles_m = 0; f.dbias = nullptr; }
    if (pd) d = *pd;
    else { d = *pf; d.tiles_m = 0; }
    if (pd && pf && (pd->M != pf->Kd || pd->Kd != pf->M || pd->Ncols != pf->Ncols || pd->mask != pf->mask)) return hipErrorInvalidValue;
    const int wgs = d.tiles_m * d.tiles_n + f.tiles_m * f.tiles_n;
    if (!bf16) return bwd32(d, f, wgs, s);
    if (f.M % 2 == 0) return f.Ncols % 2 == 0 ? bwd16<true, true>(d, f, wgs, s) : bwd16<true, false>(d, f, wgs, s);
    return f.Ncols % 2 == 0 ? bwd16<false, true>(d, f, wgs, s) : bwd16<false, false>(d, f, wgs, s);
}

}  // namespace owt
