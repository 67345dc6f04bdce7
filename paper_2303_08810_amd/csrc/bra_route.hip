// Routing rows on their own (bra_route_dev.h).
#include "bra_route_dev.h"

namespace bra {

using namespace mfma;

namespace {

template <bool VEC>
__global__ __launch_bounds__(64 * route::kWaves) void k_route_rows(const float *__restrict__ Qr, const float *__restrict__ Kr,
                                                            int ld, int32_t *__restrict__ Ir, float *__restrict__ Ar,
                                                            Dims D, int CS)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    route::route_block<VEC, true, 6>(Qr, Kr, ld, Ir, Ar, D, CS, blockIdx.x, smem);
}

}  // namespace

int route_rows(const Dims &D, const float *Qr, const float *Kr, int ld, int32_t *Ir, float *Ar_opt, hipStream_t st)
{
    if (!route::supported(D)) return BRA_ERR_UNSUPPORTED;
    const route::Plan p = route::plan(D, ld);
    static bool opted = false;
    if (!opted && p.smem > 64 * 1024) {
        if (hipFuncSetAttribute((const void *)k_route_rows<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess ||
            hipFuncSetAttribute((const void *)k_route_rows<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess)
            return BRA_ERR_LAUNCH;
        opted = true;
    }
    ProfScope ps(st, K_MFMA_ROUTE_ROWS);
    const dim3 grid((unsigned)p.blocks), threads(64 * route::kWaves);
    if (p.vec) hipLaunchKernelGGL(k_route_rows<true>, grid, threads, p.smem, st, Qr, Kr, ld, Ir, Ar_opt, D, p.CS);
    else hipLaunchKernelGGL(k_route_rows<false>, grid, threads, p.smem, st, Qr, Kr, ld, Ir, Ar_opt, D, p.CS);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace bra
