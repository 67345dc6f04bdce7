// Depth-wise convolution passes on bf16 maps (walk_tile in bra_lce_pairs.h).
#include "bra_lce_pairs.h"
#include "bra_route_dev.h"

namespace bra {
namespace lce {

namespace {

// GRAD = false: Out += LCE(In).
// GRAD = true:  Out += LCE^T(In) and the tap gradients, summed over the workgroup's tiles: Part[group][C][25].
template <bool GRAD>
__global__ __launch_bounds__(256) void k_lce_pairs(const bf16_t *__restrict__ In, const bf16_t *__restrict__ V,
                                                   const bf16_t *__restrict__ Wlce, bf16_t *__restrict__ Out, int ldo,
                                                   float *__restrict__ Part, Dims D, Tiling T, int cblocks, long tiles,
                                                   int tiles_per_wg)
{
    __shared__ __attribute__((aligned(16))) float red[GRAD ? 25 * 256 : kTapBytes / 4];
    const int block = mfma::swizzled_block(), cb = block % cblocks, c0 = 64 * cb, grp = block / cblocks;
    const long first = (long)grp * tiles_per_wg, last = min(tiles, first + tiles_per_wg);
    if (first >= tiles) return;
    const int cp = threadIdx.x % 32, slot = threadIdx.x / 32;
    TapTable &table = *(TapTable *)red;
    stage_taps<GRAD, 256>(table, Wlce, c0, D.C);
    const bool live = c0 + 2 * cp < D.C;
    const int cl = live ? 2 * cp : 0;
    u32x2 w[5][3];
    load_taps(w, table, cl);
    float acc[GRAD ? 25 : 1][2];
#pragma unroll
    for (int t = 0; t < (GRAD ? 25 : 1); ++t) acc[t][0] = acc[t][1] = 0.f;
    if (GRAD) __syncthreads();
    for (long tile = first; tile < last; ++tile) walk_tile<GRAD, true>(In, V, Out, ldo, D, T, tile, slot, c0, cl, live, w, acc);
    if (!GRAD) return;
    // the 8 slots' sums of a channel through LDS, added in a fixed order
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < (GRAD ? 25 : 1); ++t) red[t * 256 + threadIdx.x] = acc[t][v];
        __syncthreads();
        for (int e = threadIdx.x; e < 25 * 32; e += 256) {
            const int t = e / 32, ch = c0 + 2 * (e % 32) + v;
            float s = 0.f;
            for (int k = 0; k < 8; ++k) s += red[t * 256 + k * 32 + e % 32];
            if (ch < D.C) Part[((size_t)grp * D.C + ch) * 25 + 24 - t] = s;
        }
    }
}

// Out = LCE(In) beside the rows of A^r and their top-k: the routing is a chain of latencies on a few workgroups (13 us for
// 8 x 64 regions of 768 channels), and the convolution needs nothing of it.  Workgroups below route_blocks (a multiple of 8;
// those without rows leave) do the routing, the others two tiles each.  Routing, convolution in place and attention took 119.5 us
// as a layer of 2 x 200 x 300 x 64, S = 16, and 124.0 of 8 x 32 x 32 x 768; with the convolution here 113.6 and 110.
constexpr int kStoreThreads = 64 * route::kWaves;

struct StoreJob {
    const bf16_t *In, *Wlce;
    bf16_t *Out;
    Tiling T;
    int cblocks;
    long tiles;
};

__global__ __launch_bounds__(kStoreThreads, 4) void k_route_lce(const float *__restrict__ Qr, const float *__restrict__ Kr, int32_t *__restrict__ Ir,
                                                                int CS, int rows_blocks, int route_blocks, StoreJob J, Dims D)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int bi = blockIdx.x;
    if (bi < route_blocks) {
        if (bi < rows_blocks) route::route_block<true, 3>(Qr, Kr, D.C, Ir, nullptr, D, CS, bi, smem);
        return;
    }
    const int per_xcd = ((int)gridDim.x - route_blocks) / 8, block = (bi % 8) * per_xcd + (bi - route_blocks) / 8;
    const int c0 = 64 * (block % J.cblocks), cl = 2 * (threadIdx.x % 32);
    if ((long)(block / J.cblocks) * 2 >= J.tiles) return;
    TapTable &table = *(TapTable *)smem;
    stage_taps<false, kStoreThreads>(table, J.Wlce, c0, D.C);
    u32x2 w[5][3];
    load_taps(w, table, cl);
    float none[1][2];
    const long tile = (long)(block / J.cblocks) * 2 + threadIdx.x / 256;
    if (tile < J.tiles)
        walk_tile<false, false>(J.In, (const bf16_t *)nullptr, J.Out, D.C, D, J.T, tile, threadIdx.x / 32 % 8, c0, cl, true, w, none);
}

}  // namespace

// Qr = NULL: the convolution alone.  BRA_ERR_UNSUPPORTED, with nothing enqueued, for maps too wide for its strips.
int route_rows_lce_bf16(const Dims &D, const float *Qr, const float *Kr, int32_t *Ir, const bf16_t *V, const bf16_t *Wlce, bf16_t *O,
                        hipStream_t st)
{
    StoreJob J = {V, Wlce, O, Tiling{}, D.C / 64, 0};
    J.T = tiling(D, D.C, 1536 / J.cblocks, J.tiles);
    const long lce_blocks = ((J.tiles + 1) / 2 * J.cblocks + 7) / 8 * 8;
    if (D.C % 64 || !route::supported(D) || !offsets_fit(D, J.T, D.C) || lce_blocks > 0x3fffffffL) return BRA_ERR_UNSUPPORTED;
    const route::Plan p = route::plan(D, D.C);
    const int rb = Qr ? p.blocks : 0, route_blocks = (rb + 7) / 8 * 8;
    const size_t smem = std::max(rb ? p.smem : 0, kTapBytes);
    static bool opted = false;
    if (!opted && smem > 64 * 1024) {
        if (hipFuncSetAttribute((const void *)k_route_lce, hipFuncAttributeMaxDynamicSharedMemorySize, mfma::kMaxLds) != hipSuccess) return BRA_ERR_LAUNCH;
        opted = true;
    }
    ProfScope ps(st, rb ? K_MFMA_ROUTE_ROWS : K_MFMA_LCE_ADD);
    hipLaunchKernelGGL(k_route_lce, dim3((unsigned)(route_blocks + lce_blocks)), dim3(kStoreThreads), smem, st, Qr, Kr, Ir, p.CS, rb, route_blocks, J, D);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// Maps so wide that not even strips of 5 rows fit (119 million values in a row) take the kernels of bra_lce_dev.h, whose
// addresses are 64-bit throughout.
int lce_add_bf16(const Dims &D, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, int ldo, int kernel_id, hipStream_t st)
{
    const int cblocks = (D.C + 63) / 64;
    long tiles;
    const Tiling T = tiling(D, ldo, 1536 / cblocks, tiles);
    const long blocks = tiles * cblocks;
    if (!offsets_fit(D, T, ldo)) return launch_lce<bf16_t, bf16_t>(D, V, D.C, Wlce, O, ldo, kernel_id, st);
    if (D.C % 2 || ldo % 2 || blocks > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_pairs<false>, dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, st, V, (const bf16_t *)nullptr,
                       Wlce, O, ldo, (float *)nullptr, D, T, cblocks, tiles, 1);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

namespace {

// About 768 workgroups (three per compute unit), each with the tiles of one group.
constexpr int kGradSlots = 768;

Tiling grad_plan(const Dims &D, int lddv, long &tiles, int &per_wg, int &groups)
{
    const int cblocks = (D.C + 63) / 64;
    const long want = std::max(1, kGradSlots / cblocks);
    const Tiling T = tiling(D, lddv, want, tiles);
    per_wg = (int)((tiles + want - 1) / want);
    groups = (int)((tiles + per_wg - 1) / per_wg);
    return T;
}

LcePlan wide_grad_plan(const Dims &D) { return lce_plan(D, kGradSlots, 8); }      // 8 columns per workgroup: two channels per thread

}  // namespace

int lce_grad_groups_bf16(const Dims &D, int lddv)
{
    long tiles;
    int per_wg, groups;
    return offsets_fit(D, grad_plan(D, lddv, tiles, per_wg, groups), lddv) ? groups : wide_grad_plan(D).groups;
}

int lce_grad_bf16(const Dims &D, const bf16_t *dO, const bf16_t *V, const bf16_t *Wlce, bf16_t *dV, int lddv, float *Part,
                  int kernel_id, hipStream_t st)
{
    const int cblocks = (D.C + 63) / 64;
    long tiles;
    int per_wg, groups;
    const Tiling T = grad_plan(D, lddv, tiles, per_wg, groups);
    if (D.C % 2 || lddv % 2) return BRA_ERR_UNSUPPORTED;
    if (!offsets_fit(D, T, lddv)) {
        ProfScope ps(st, kernel_id);
        return launch_lce_grad<bf16_t, bf16_t>(D, wide_grad_plan(D), dO, V, D.C, Wlce, dV, lddv, Part, st);
    }
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_pairs<true>, dim3((unsigned)((groups * cblocks + 7) / 8 * 8)), dim3(256), 0, st, dO, V, Wlce, dV,
                       lddv, Part, D, T, cblocks, tiles, per_wg);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace lce
}  // namespace bra
