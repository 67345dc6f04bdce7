// Depth-wise convolution passes on bf16 maps (walk_tile in bra_lce_pairs.h).
#include "bra_lce_pairs.h"
#include "bra_route_dev.h"

namespace bra {
namespace lce {

namespace {

__global__ __launch_bounds__(256) void k_lce_add(Job J, Dims D)
{
    __shared__ __attribute__((aligned(16))) float lds[job_bytes<false>() / 4];
    job_block<false, true>(J, D, mfma::swizzled_block(), lds);
}

// dV += LCE^T(dO) with the tap gradients, and O += LCE(V), in one launch (two launches took 41.6 us for 64 x 14 x 14 x 384, this
// one 26.6).
__global__ __launch_bounds__(256) void k_lce_backward(Job grad, Job add, int grad_blocks, Dims D)
{
    __shared__ __attribute__((aligned(16))) float lds[job_bytes<true>() / 4];
    const int bi = blockIdx.x;
    if (bi < grad_blocks) job_block<true, true>(grad, D, mfma::swizzled(bi, grad_blocks), lds);
    else job_block<false, true>(add, D, mfma::swizzled(bi - grad_blocks, (int)gridDim.x - grad_blocks), lds);
}

// LCE(In) in float32 (halves in Out and Low) beside the rows of A^r and their top-k: the routing is a chain of latencies on a few workgroups (13 us for
// 8 x 64 regions of 768 channels), and the convolution needs nothing of it.  Workgroups below route_blocks (a multiple of 8;
// those without rows leave) do the routing, the others two tiles each.  Figures for
// whole layers stand at the call.
constexpr int kStoreThreads = 64 * route::kWaves;

__global__ __launch_bounds__(kStoreThreads, 4) void k_route_lce(const float *__restrict__ Qr, const float *__restrict__ Kr, int32_t *__restrict__ Ir,
                                                                int CS, int rows_blocks, int route_blocks, Job J, Dims D)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int bi = blockIdx.x;
    if (bi < route_blocks) {
        if (bi < rows_blocks) route::route_block<true, false, 3>(Qr, Kr, D.C, Ir, nullptr, D, CS, bi, smem);
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
    const long tile = (long)(block / J.cblocks) * 2 + __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
    if (tile < J.tiles)
        walk_tile<false, false>(J.In, (const bf16_t *)nullptr, J.Out, J.Low, D.C, D, J.T, tile, threadIdx.x / 32 % 8, c0, cl, true, w, none);
}

}  // namespace

namespace {

Job plain_job(const Dims &D, const bf16_t *In, const bf16_t *Wlce, bf16_t *Out, int ldo, int beside)
{
    Job J = {In, nullptr, Wlce, Out, nullptr, nullptr, ldo, (D.C + 63) / 64, 1, 0, Tiling{}};
    J.T = forward_tiling(D, ldo, J.cblocks, beside, J.tiles);
    return J;
}

// Workgroups with tap gradients, each with the tiles of one group: two per compute unit, so that the third place is left to
// the kernel beside them (query side of 64 x 56 x 56 x 64, k = 1, with the pass in front: 55.4 us, 57.8 with three per compute
// unit; the two passes alone for 64 x 14 x 14 x 384: 26.6 and 30.3).  Workgroups of the other pass, behind the key side: three
// per compute unit (28 x 28 x 128 at B = 64: 40 us, 42 with one tile each; two per compute unit: 41, but 65 for 57 at 64 channels).
constexpr int kGradSlots = 512, kAddSlots = 768;

// Strips no lower than it takes for this many tiles of 64 channels: a lower strip reads its four rows of window again.  Whole gradient, us, for
// 256, 320, 360 and 480: 16 x 28 x 28 x 192 72.6, 71.8, 72.0, 75.7; 9 x 28 x 42 x 384 120.9, 121.0, 124.5, 124.7; 8 x 56 x 56 x 64 71.0, 69.7, 69.6, 69.7.
constexpr int kEnoughBlocks = 320;

Job job(const Dims &D, const bf16_t *In, const bf16_t *V, const bf16_t *Wlce, bf16_t *Out, int ldo, float *Part, int workgroups)
{
    Job J = {In, V, Wlce, Out, nullptr, Part, ldo, (D.C + 63) / 64, 1, 0, Tiling{}};
    const long want = std::max(1, workgroups / J.cblocks);
    J.T = even_tiling(D, ldo, std::max(1, kEnoughBlocks / J.cblocks), J.tiles);
    J.per_wg = (int)((J.tiles + want - 1) / want);
    return J;
}

LcePlan wide_grad_plan(const Dims &D) { return lce_plan(D, 768, 8); }      // 8 columns per workgroup: two channels per thread

}  // namespace

BackwardJobs backward_jobs(const Dims &D, const bf16_t *dO, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, bf16_t *dV, bf16_t *dK, int lddv, float *Part)
{
    BackwardJobs L;
    L.grad = job(D, dO, V, Wlce, dV, lddv, Part, kGradSlots);
    L.grad.Low = dK;
    L.add = job(D, V, nullptr, Wlce, O, D.C, nullptr, kAddSlots);
    L.fit = offsets_fit(D, L.grad.T, lddv) && offsets_fit(D, L.add.T, D.C);
    const long values = (long)D.B * D.N * D.C;
    L.beside = L.fit && (values <= 14L << 20 || (D.n > 96 && D.C <= 128 && values <= 28L << 20));
    return L;
}

// Qr = NULL: the convolution alone.  BRA_ERR_UNSUPPORTED, with nothing enqueued, for maps too wide for its strips.
int route_rows_lce_bf16(const Dims &D, const float *Qr, const float *Kr, int32_t *Ir, const bf16_t *V, const bf16_t *Wlce, bf16_t *O,
                        bf16_t *Low, hipStream_t st)
{
    const route::Plan p = route::plan(D, D.C);
    const int rb = Qr ? p.blocks : 0, route_blocks = (rb + 7) / 8 * 8;
    Job J = plain_job(D, V, Wlce, O, D.C, route_blocks);
    J.Low = Low;
    const long lce_blocks = ((J.tiles + 1) / 2 * J.cblocks + 7) / 8 * 8;
    if (D.C % 64 || !route::supported(D) || !offsets_fit(D, J.T, D.C) || lce_blocks > 0x3fffffffL) return BRA_ERR_UNSUPPORTED;
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

// Maps so wide that not even strips of 4 rows fit (134 million values in a row) take the kernels of bra_lce_dev.h, whose
// addresses are 64-bit throughout.
int lce_add_bf16(const Dims &D, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, int ldo, int kernel_id, hipStream_t st)
{
    const Job J = plain_job(D, V, Wlce, O, ldo, 0);
    if (!offsets_fit(D, J.T, ldo)) return launch_lce<bf16_t>(D, V, D.C, Taps(Wlce), O, ldo, kernel_id, st);
    if (D.C % 2 || ldo % 2 || J.blocks() > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_add, dim3((unsigned)J.blocks()), dim3(256), 0, st, J, D);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

int lce_grad_groups_bf16(const Dims &D, int lddv)
{
    const BackwardJobs L = backward_jobs(D, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, lddv, nullptr);
    return L.fit ? (int)L.grad.groups() : wide_grad_plan(D).groups;
}

int lce_backward_bf16(const Dims &D, const BackwardJobs &L, int kernel_id, hipStream_t st)
{
    const Job &G = L.grad, &A = L.add;
    if (D.C % 2 || G.ldo % 2) return BRA_ERR_UNSUPPORTED;
    if (!L.fit) {
        const int rc = launch_lce<bf16_t>(D, A.In, D.C, Taps(A.Wlce), A.Out, A.ldo, kernel_id, st);
        if (rc != BRA_OK) return rc;
        ProfScope ps(st, kernel_id);
        return launch_lce_grad<bf16_t>(D, GradJob<bf16_t>{G.In, G.V, Taps(G.Wlce), G.Out, G.Part, D.C, G.ldo, wide_grad_plan(D)}, st);
    }
    if (G.blocks() + A.blocks() > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_backward, dim3((unsigned)(G.blocks() + A.blocks())), dim3(256), 0, st, G, A, (int)G.blocks(), D);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace lce
}  // namespace bra
