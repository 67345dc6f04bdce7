// Float32 kernel family: float32 arithmetic, any valid shape.
//
// Used for float32 tensors and for shapes the bf16 matrix-core kernels are not built
// for.  All intermediates (Q, K, V, attention output) are kept in float32 in the
// workspace, whatever the storage type of X and Y.  The steps follow Sec. 3.2:
// projection (Eq. 3), region pooling + affinity (Eq. 4), top-k (Eq. 5), routed
// attention straight from the index (Eq. 6-7, no gathered tensor), LCE, W^o (Eq. 2).
// Products run on the float32 matrix-core instruction (bra_f32_dev.h, bra_route.hip); heads wider
// than 64 channels and the block's LayerNorms are scalar kernels.
// Region pooling uses mean(X^r) W = mean(X^r W), which is exact in real arithmetic
// (the mean is linear; same argument as Appendix A).
#include "bra_f32_heads_dev.h"
#include "bra_route_dev.h"

#include <algorithm>
#include <type_traits>

#include <math.h>

namespace bra {

namespace {

constexpr int kWave = 64;
constexpr int kMaxRegions = 1024;   // what route_rows takes
constexpr int kAttnChunk = 1024;    // keys per online-softmax chunk
constexpr int kAttnMaxD = 256;      // head width limit of the generic attention kernel

// ---------------------------------------------------------------------------
// Routed attention for wider heads, one workgroup (4 wavefronts) per (b, region i, head).  Each
// wavefront owns one query at a time and runs an online softmax over the k n keys
// of regions Ir[b, i, :] in chunks; keys and values are read in place from the
// projected map by index.  QKV is [B, N, 3C] float32 (q | k | v per token).
__global__ __launch_bounds__(256) void gen_attention(const float *__restrict__ QKV,
                                                     const int32_t *__restrict__ Ir,
                                                     float *__restrict__ O, Dims D, float scale, bool adds)
{
    __shared__ float qs[4][kAttnMaxD];
    __shared__ float sc[4][kAttnChunk];
    __shared__ int tk[4][kAttnChunk];
    extern __shared__ int regs[];  // k routed regions

    const int hd = blockIdx.x % D.heads;
    const int i = (blockIdx.x / D.heads) % D.R;
    const int b = blockIdx.x / (D.heads * D.R);
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int C3 = 3 * D.C;
    const float *img = QKV + (size_t)b * D.N * C3;

    for (int p = threadIdx.x; p < D.k; p += blockDim.x) regs[p] = region_index(Ir[((size_t)b * D.R + i) * D.k + p], D.R);
    __syncthreads();

    const int y0 = (i / D.S) * D.rh, x0 = (i % D.S) * D.rw;
    const int iters = (D.n + 3) / 4;
    for (int it = 0; it < iters; ++it) {
        const int s = it * 4 + wave;
        const bool active = s < D.n;
        int qtok = 0;
        if (active) {
            qtok = (y0 + s / D.rw) * D.W + x0 + s % D.rw;
            for (int c = lane; c < D.d; c += kWave) qs[wave][c] = img[(size_t)qtok * C3 + hd * D.d + c];
        }
        float m = -INFINITY, l = 0.f;
        float acc[kAttnMaxD / kWave];
        for (int t = 0; t < kAttnMaxD / kWave; ++t) acc[t] = 0.f;
        __syncthreads();
        for (int c0 = 0; c0 < D.kn; c0 += kAttnChunk) {
            const int cn = min(kAttnChunk, D.kn - c0);
            float lm = -INFINITY;
            if (active) {
                for (int u = lane; u < cn; u += kWave) {
                    const int g = c0 + u;
                    const int j = regs[g / D.n], slot = g % D.n;
                    const int tok = ((j / D.S) * D.rh + slot / D.rw) * D.W + (j % D.S) * D.rw + slot % D.rw;
                    const float *kr = img + (size_t)tok * C3 + D.C + hd * D.d;
                    float a = 0.f;
                    for (int c = 0; c < D.d; ++c) a = fmaf(qs[wave][c], kr[c], a);
                    a *= scale;
                    sc[wave][u] = a;
                    tk[wave][u] = tok;
                    lm = fmaxf(lm, a);
                }
            }
            for (int off = 32; off >= 1; off >>= 1) lm = fmaxf(lm, __shfl_xor(lm, off, kWave));
            const float m_new = fmaxf(m, lm);
            const float corr = (m == -INFINITY) ? 0.f : expf(m - m_new);
            float ls = 0.f;
            if (active) {
                for (int u = lane; u < cn; u += kWave) {
                    float pv = expf(sc[wave][u] - m_new);
                    sc[wave][u] = pv;
                    ls += pv;
                }
            }
            for (int off = 32; off >= 1; off >>= 1) ls += __shfl_xor(ls, off, kWave);
            l = l * corr + ls;
            m = m_new;
            __syncthreads();
            if (active) {
                for (int t = 0; t < kAttnMaxD / kWave; ++t) {
                    const int c = lane + t * kWave;
                    if (c < D.d) {
                        float a = acc[t] * corr;
                        for (int u = 0; u < cn; ++u)
                            a = fmaf(sc[wave][u], img[(size_t)tk[wave][u] * C3 + 2 * D.C + hd * D.d + c], a);
                        acc[t] = a;
                    }
                }
            }
            __syncthreads();
        }
        if (active) {
            for (int t = 0; t < kAttnMaxD / kWave; ++t) {
                const int c = lane + t * kWave;
                if (c >= D.d) continue;
                float *o = O + ((size_t)b * D.N + qtok) * D.C + hd * D.d + c;
                *o = adds ? *o + acc[t] / l : acc[t] / l;
            }
        }
    }
}

struct GenericWs {
    float *qkv, *o, *xr, *qk;        // qk: Q^r | K^r, interleaved rows of 2C
    int32_t *ir;
    size_t bytes;
};

GenericWs carve(const Dims &D, void *ws)
{
    GenericWs w;
    char *p = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *q = p ? p + off : nullptr; off += align256(bytes); return q; };
    const size_t tok = (size_t)D.B * D.N, reg = (size_t)D.B * D.R;
    w.qkv = (float *)take(tok * 3 * D.C * sizeof(float));
    w.o = (float *)take(tok * D.C * sizeof(float));
    w.xr = (float *)take(reg * D.C * sizeof(float));
    w.qk = (float *)take(reg * 2 * D.C * sizeof(float));
    w.ir = (int32_t *)take(reg * D.k * sizeof(int32_t));
    w.bytes = off;
    return w;
}

constexpr int kAttnF32MaxD = 64;    // head width up to which attention runs on the matrix cores

bool launched() { return hipGetLastError() == hipSuccess; }

// 64-column tiles with a float32 matrix, where the matrix cores are the bound and nothing may be left of a tile (50176 x 64 x
// 192: 19.4 us, 23.7 with 128 columns; whole gradient of 3136 x 384: 199 and 205, of 6272 x 128 the same); with a bf16 one where
// wider ones would leave the chip under-filled (else memory is the bound: 42336 x 96 x 288 takes 18.5 with narrow tiles, 17.1).
// The other tile.
template <typename TB>
constexpr int kWideBN = std::is_same<TB, float>::value ? 64 : 128;

template <typename TB>
bool narrow_tiles(long M, int N, int N1 = 0)
{
    const long mt = (M + f32::kGemmBM - 1) / f32::kGemmBM;
    return std::is_same<TB, float>::value || N <= 64 || mt * ((N + 127) / 128 + (N1 + 127) / 128) < 512;
}

// Workgroups of so many tiles: those with a bf16 matrix are dealt out by XCD.
template <typename TB>
long tile_blocks(long tiles) { return std::is_same<TB, float>::value ? tiles : (tiles + 7) / 8 * 8; }

// Float32 products of few rows (N1: columns of a second one over the same rows) by split_tile: where the tiles of 64 x 64 leave half of the chip
// idle or more. Those take 0.75 us for 32 of the contraction however few they are; the split ones read both operands two to four times as often,
// which shows from 128 of the others on, and earlier where the contraction is short. Tiles of 64 / split (us, whole calls): 24 tiles, 1 x 7 x 7 x 512
// 46.1 / 24.4; 72, 2 x 8 x 8 x 768 63.2 / 42.1; 112, 2 x 14 x 14 x 512's gradients 90.5 / 74.0; 80, 3 x 14 x 14 x 256 33.4 / 29.7; 12 rows of K = 3 C, gradients
// of 1 x 7 x 7 x 768 131.5 / 83.8; beyond: 216, 7 x 7 x 7 x 768 67.7 / 79.1; 117 of K = 192, 1 x 28 x 28 x 192 26.7 / 27.9, 104 of K = 128, gradients of 1 x
// 28 x 28 x 128 36.4 / 38.5, 60 of K = 128, 1 x 40 x 24 x 128 24.4 / 26.1 (36, 1 x 24 x 24 x 128 23.3 / 22.9).
bool splits(long M, int N, int K, int N1 = 0)
{
    return K >= 64 && N % 32 == 0 && N1 % 32 == 0 && K % 16 == 0 && (M + 63) / 64 * ((N + 63) / 64 + (N1 + 63) / 64) <= (K >= 256 ? 128 : K > 128 ? 64 : 40);
}

// Rows of its tiles, 16 or 32: by the rounds of 256 workgroups (2 x 8 x 8 x 768 42.1 / 47.1 us), the larger where they take the same, which read less
// (3 x 14 x 14 x 256 29.8 / 29.1, 4 x 7 x 14 x 512's block 107 / 104).  A value's sums are the same with both.
int split_rows(long M, int N, int N1 = 0)
{
    auto rounds = [&](int rows) { return ((M + rows - 1) / rows * ((N + N1) / 32) + 255) / 256; };
    return rounds(16) < 2 * rounds(32) ? 16 : 32;
}

// One or two products in one launch (J1: NULL for one).
template <bool BT, bool VEC, typename TA, typename TB, typename TO>
int launch_gemm_vec(const f32::GemmJob<TA, TB, TO> &J0, const f32::GemmJob<float, TB, float> *J1, hipStream_t st)
{
    const bool narrow = narrow_tiles<TB>(J0.M, J0.N);
    const int bn = narrow ? 64 : 128;
    auto blocks = [&](long M, int N) { return tile_blocks<TB>((M + f32::kGemmBM - 1) / f32::kGemmBM * ((N + bn - 1) / bn)); };
    const long b0 = blocks(J0.M, J0.N), b1 = J1 ? blocks(J1->M, J1->N) : 0;
    if (b0 + b1 > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    const f32::GemmJob<float, TB, float> none = {};
    const f32::GemmJob<float, TB, float> &j1 = J1 ? *J1 : none;
    if (narrow)
        hipLaunchKernelGGL((f32::k_gemm<BT, VEC, 64, TA, TB, TO>), dim3((unsigned)(b0 + b1)), dim3(256), 0, st, J0, j1, (int)b0);
    else
        hipLaunchKernelGGL((f32::k_gemm<BT, VEC, kWideBN<TB>, TA, TB, TO>), dim3((unsigned)(b0 + b1)), dim3(256), 0, st, J0, j1, (int)b0);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

// may_split: false for a product that is the second one of a launch elsewhere, where it is summed in one chain, and has to come out with the same bits.
template <bool BT, typename TA, typename TB, typename TO>
int launch_gemm(const f32::GemmJob<TA, TB, TO> &J0, const f32::GemmJob<float, TB, float> *J1, hipStream_t st, bool may_split = true)
{
    auto quads = [](int a, int b, int c, int d, int e) { return (a | b | c | d | e) % 4 == 0; };
    const bool vec = quads(J0.lda, J0.ldb, J0.ldo, J0.N, J0.K) && (!J1 || quads(J1->lda, J1->ldb, J1->ldo, J1->N, J1->K));
    if constexpr (!BT && std::is_same<TA, float>::value && std::is_same<TB, float>::value && std::is_same<TO, float>::value) {
        if (vec && !J1 && may_split && splits(J0.M, J0.N, J0.K)) {
            const int rows = split_rows(J0.M, J0.N);
            const dim3 grid((unsigned)((J0.M + rows - 1) / rows * (J0.N / 32)));
            if (rows == 16) hipLaunchKernelGGL((f32::k_gemm_split<false, 1>), grid, dim3(512), 0, st, J0);
            else hipLaunchKernelGGL((f32::k_gemm_split<false, 2>), grid, dim3(512), 0, st, J0);
            return launched() ? BRA_OK : BRA_ERR_LAUNCH;
        }
    }
    return vec ? launch_gemm_vec<BT, true>(J0, J1, st) : launch_gemm_vec<BT, false>(J0, J1, st);
}

template <typename T>
void launch_pool(const Dims &D, const T *X, float *Xr, hipStream_t st)
{
    int sub = 1;                                               // lanes per (region, 4-channel chunk)
    while (sub < 16 && 4 * sub <= D.n) sub *= 2;
    const long items = (long)D.B * D.R * ((D.C + 3) / 4) * sub;
    const dim3 grid((unsigned)((items + 255) / 256));
    ProfScope ps(st, K_GEN_POOL);
    if (D.C % 4 == 0) hipLaunchKernelGGL((f32::k_pool<T, true>), grid, dim3(256), 0, st, X, Xr, D, sub);
    else hipLaunchKernelGGL((f32::k_pool<T, false>), grid, dim3(256), 0, st, X, Xr, D, sub);
}

// Q^r | K^r = Xr [Wq | Wk]: columns 0 .. 2C - 1 of Wqkv, interleaved rows of 2C.
template <typename T>
f32::GemmJob<float, T, float> region_job(const Dims &D, const T *Wqkv, const GenericWs &w)
{
    return {w.xr, Wqkv, w.qk, (long)D.B * D.R, D.C, 3 * D.C, 2 * D.C, 2 * D.C, D.C, nullptr, nullptr, 0};
}

// The means of Q and K out of the token projection, whose tiles go region by region: a pooling pass and a region-level product less for
// bra_forward.  bra_route, which has to decide on the same bits, projects all tokens for it; the lines lie about where that takes as
// long.  bra_forward before -> now / bra_route (us): 4 x 14 x 14 x 256 38.3 -> 35.9 / 18.8 -> 15.7, 2 x 64 x 64 x 128 49.5 -> 44.8, 1 x 21 x 21 x 768 79.3 -> 65.7, 50 x 28
// x 28 x 96 bf16 74.7 -> 69.7 / 17.6 -> 15.2.  bra_route pays more where tiles have idle rows: 2 x 35 x 35 x 192 (25 tokens per region) 41.4 -> 38.8 / 16.0 -> 17.3, 12 x 56 x
// 48 x 96 bf16, S = 8 (42) 74.1 -> 72.6 / 14.0 -> 15.9, 21 x 35 x 35 x 64 (25) 14.3 -> 16.5; bra_forward where they make it two
// rounds of workgroups for one: 1 x 35 x 35 x 256, k = 1 37.2 -> 39.0 / 17.9 -> 15.5.
// float32, by tiles of bra_route's product times C, bra_route: 56 thousand (C = 192) 17.1 -> 16.6, 66 (128) 15.5 -> 14.1, 72 (128) 16.9 -> 17.0, 88 (96, 36 tokens) 14.1
// -> 17.0, 100 (64) 15.0 -> 18.4; 312 tiles of C = 768 36.0 -> 44.2, 168 35.5 -> 32.2.  bf16, by millions of values: 3.1 (C = 160) 17.4 -> 14.4, 5.5 (96) 28.8 -> 27.8, 5.5
// (288) 25.2 -> 27.6, 9.2 (160) 24.4 -> 25.9, regions of 4 tokens 9.2 47.3 -> 44.7.
bool means_from_projection(const Dims &D)
{
    const long values = (long)D.B * D.N * D.C;
    if (D.n > f32::kGemmBM || D.C % 4 != 0 || (long)D.B * D.N > 0x7fffffffL) return false;
    if (D.dtype == BRA_BF16) return values <= (D.n <= 4 ? 10L << 20 : 4L << 20);
    const long per = f32::kGemmBM / D.n, tiles = ((long)D.B * D.R + per - 1) / per * ((2L * D.C + 63) / 64);
    return D.n == 1 || tiles <= 256 || tiles * D.C <= (D.n <= 4 ? 80000 : 66000);
}

// Out: Q | K | V of all tokens, or NULL for Q^r | K^r alone.
template <typename T>
int launch_gemm_means(const Dims &D, const T *X, const T *Wqkv, float *Out, const GenericWs &w, hipStream_t st)
{
    const int C = D.C, N = Out ? 3 * C : 2 * C, per = f32::kGemmBM / D.n;
    const f32::GemmJob<T, T, float> J = {X, Wqkv, Out, (long)D.B * D.N, C, 3 * C, 3 * C, N, C, nullptr, nullptr, 0};
    const f32::MeansJob means = {w.qk, 2 * C, D.B * D.R, D.R, D.S, D.n, D.rh, D.rw, 1.0f / D.n, 1.0f / D.R, 1.0f / D.S, 1.0f / D.rw};
    if constexpr (std::is_same<T, float>::value) {
        // by the columns of Q and K for both callers: bra_route decides on the same bits as bra_forward
        if (D.n <= 32 && C % 32 == 0 && splits(J.M, 2 * C, C)) {
            const int rows = D.n <= 16 ? split_rows(J.M, 3 * C) : 32, each = rows / D.n;
            const dim3 grid((unsigned)(((long)D.B * D.R + each - 1) / each * (N / 32)));
            if (rows == 16) hipLaunchKernelGGL(f32::k_gemm_means_split<1>, grid, dim3(512), 0, st, J, means);
            else hipLaunchKernelGGL(f32::k_gemm_means_split<2>, grid, dim3(512), 0, st, J, means);
            return launched() ? BRA_OK : BRA_ERR_LAUNCH;
        }
    }
    const long row_tiles = ((long)D.B * D.R + per - 1) / per;
    const bool narrow = narrow_tiles<T>(row_tiles * f32::kGemmBM, N);
    const int bn = narrow ? 64 : 128;
    const long blocks = tile_blocks<T>(row_tiles * ((N + bn - 1) / bn));
    if (blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    if (narrow) hipLaunchKernelGGL((f32::k_gemm_means<64, T>), dim3((unsigned)blocks), dim3(256), 0, st, J, means);
    else hipLaunchKernelGGL((f32::k_gemm_means<kWideBN<T>, T>), dim3((unsigned)blocks), dim3(256), 0, st, J, means);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

// Routing on its own: region means, their projection, rows of A^r and top-k.  The arithmetic of every entry is that
// of forward_t, so both give the same index.
template <typename T>
int launch_route(const Dims &D, const T *X, const T *Wqkv, int32_t *Ir, float *Ar_opt, const GenericWs &w, hipStream_t st)
{
    if (means_from_projection(D)) {
        {
            ProfScope ps(st, K_GEN_REGION_QK);
            const int rc = launch_gemm_means<T>(D, X, Wqkv, nullptr, w, st);
            if (rc != BRA_OK) return rc;
        }
        return route_rows(D, w.qk, w.qk + D.C, 2 * D.C, Ir, Ar_opt, st);
    }
    launch_pool<T>(D, X, w.xr, st);
    {
        ProfScope ps(st, K_GEN_REGION_QK);
        // beside Q, K and V in forward_t
        const int rc = launch_gemm<false>(region_job<T>(D, Wqkv, w), (const f32::GemmJob<float, T, float> *)nullptr, st, false);
        if (rc != BRA_OK) return rc;
    }
    return route_rows(D, w.qk, w.qk + D.C, 2 * D.C, Ir, Ar_opt, st);
}

// The rows of A^r and their top-k, and O = LCE(V) in the same launch: the routing keeps few compute units busy, with a chain
// of latencies, and the convolution needs nothing of it.  Workgroups below route_blocks (a multiple of 8; those without
// rows leave) do the routing.  Layer of 16 x 56 x 56 x 64 float32: 77 us with the two apart, 66.7; 4 x 14 x 14 x 256: 45 and 39.
constexpr int kRouteThreads = 64 * route::kWaves;

template <bool VEC>
__global__ __launch_bounds__(kRouteThreads, 4) void k_route_lce(const float *__restrict__ Qr, const float *__restrict__ Kr, int ld,
                                                                int32_t *__restrict__ Ir, int CS, int rows_blocks, int route_blocks,
                                                                lce::AddJob<float> J, Dims D)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int block = (int)blockIdx.x - route_blocks;
    if (block >= 0) lce::lce_block<VEC ? 2 : 1, false, kRouteThreads>(J, D, mfma::swizzled(block, (int)gridDim.x - route_blocks), smem);
    else if ((int)blockIdx.x < rows_blocks) route::route_block<VEC, true, 3>(Qr, Kr, ld, Ir, nullptr, D, CS, blockIdx.x, smem);
}

// added: O holds LCE(V) (not for maps that lce_block does not take).
int launch_route_lce(const Dims &D, const GenericWs &w, const lce::Taps &taps, int32_t *Ir, bool &added, hipStream_t st)
{
    const int C = D.C;
    const route::Plan p = route::plan(D, 2 * C);
    const lce::AddJob<float> J = lce::add_job<float>(D, w.qkv + 2 * C, 3 * C, taps, w.o, C, p.vec ? 2 : 1, kRouteThreads);
    added = J.blocks > 0;
    if (!added) return route_rows(D, w.qk, w.qk + C, 2 * C, Ir, nullptr, st);
    if (!route::supported(D)) return BRA_ERR_UNSUPPORTED;
    const int route_blocks = (p.blocks + 7) / 8 * 8;
    const size_t smem = std::max(p.smem, (size_t)25 * 64 * sizeof(float));
    if ((long)route_blocks + J.blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    static bool opted = false;
    if (!opted && smem > 64 * 1024) {
        if (hipFuncSetAttribute((const void *)k_route_lce<true>, hipFuncAttributeMaxDynamicSharedMemorySize, mfma::kMaxLds) != hipSuccess ||
            hipFuncSetAttribute((const void *)k_route_lce<false>, hipFuncAttributeMaxDynamicSharedMemorySize, mfma::kMaxLds) != hipSuccess)
            return BRA_ERR_LAUNCH;
        opted = true;
    }
    ProfScope ps(st, K_MFMA_ROUTE_ROWS);
    const dim3 grid((unsigned)(route_blocks + J.blocks)), threads(kRouteThreads);
    if (p.vec) hipLaunchKernelGGL(k_route_lce<true>, grid, threads, smem, st, w.qk, w.qk + C, 2 * C, Ir, p.CS, p.blocks, route_blocks, J, D);
    else hipLaunchKernelGGL(k_route_lce<false>, grid, threads, smem, st, w.qk, w.qk + C, 2 * C, Ir, p.CS, p.blocks, route_blocks, J, D);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

// Query tiles of a region over workgroups: four per workgroup, or up to eight in one or more equal ones where that leaves a fifth
// fewer wavefronts (5 tiles: with four a second workgroup for the last one holds its place as long as the first;
// 17 x 49 x 70 x 96, k = 13: 441 -> 373 us)
struct TileSplit {
    int each, groups;
};

TileSplit split_tiles(int tiles, int least)
{
    const int quads = (tiles + 3) / 4, groups = (tiles + 7) / 8, even = std::max(least, (tiles + groups - 1) / groups);
    return 5 * groups * even <= 4 * 4 * quads ? TileSplit{even, groups} : TileSplit{4, quads};
}

// Workgroups of an image and head group on one XCD, or the head groups of a region on different ones.  The first reads an image's rows into
// one L2 instead of all; but of few images it leaves nothing to save where a region reads most of them, and the workgroups of an XCD
// then ask for the same lines at the same time.  Layer with a given index, us, apart / by image: float32 24 x 16 x 16 x 64, S = 8, k = 16 36.9 / 30.8,
// 4 x 24 x 32 x 128, S = 8, k = 4 33.9 / 30.5, 2 x 56 x 48 x 96, S = 8, k = 24 79.1 / 75.7; bf16 12 x 24 x 32 x 96, S = 8, k = 4 36.6 / 27.8; against that
// float32 1 x 35 x 35 x 256, k = 40 69.6 / 78.2, 1 x 49 x 42 x 128, k = 16 47.2 / 50.0, 1 x 14 x 14 x 768, k = 49 75.2 / 78.4, 2 x 35 x 35 x 192, k = 40
// 90.0 / 93.0.  Left on the wrong side: 4 x 21 x 28 x 128, k = 49 61.9 / 67.0.
bool attention_by_image(const Dims &D, int hgroups)
{
    return D.B >= 4 || (long)D.B * hgroups >= 8 || 6L * D.k <= D.R || (D.B >= 2 && 8L * D.k <= 5L * D.R);
}

// The gradients: a key region's workgroup goes over all that chose it, so that an XCD with a part of a pair has more or less work than
// the others, by chance; with a pair or more each, or many workgroups, that evens out.  us, apart / by image: float32 6 x 32 x 32 x 128, S = 8, k = 4
// 89.4 / 84.8, bf16 64 x 28 x 28 x 96, k = 16 677 / 641, 1 x 192 x 192 x 96, S = 16, k = 4 790 / 767; against that bf16 1 x 56 x 84 x 96, k = 3 120.4 / 132.2, 1 x
// 112 x 96 x 96, S = 16, k = 16 328.5 / 362.3, float32 1 x 48 x 48 x 192, S = 8, k = 2 82.6 / 88.7, 2 x 40 x 104 x 96, S = 8, k = 1 108.1 / 115.1.  Of one or
// two head groups neither is the better one on average (0.90 to 1.05) until a region reads most of its image (2 x 21 x 21 x 256, k = 49
// 156.8 / 164.0).  With a head for one, two or four wavefronts 0.96 to 1.02: bf16 4 x 28 x 28 x 96, k = 2 46.2 / 44.1, float32 14 x 28 x 28 x 128, k = 4 108.6 / 107.5, 4 x 35 x 35 x 192, k = 2
// 104.5 / 102.5; against that 6 x 28 x 28 x 128, k = 12 89.1 / 90.9, 6 x 28 x 28 x 64, k = 4 47.0 / 47.7.
bool gradients_by_image(const Dims &D, int hgroups, long workgroups)
{
    return (long)D.B * hgroups >= 8 || workgroups >= 2048 || (hgroups <= 2 && 2L * D.k <= D.R);
}

template <int DP, int HPW, bool VEC>
int launch_attention_t(const Dims &D, const float *qkv, const int32_t *Ir, float *o, bool adds, hipStream_t st)
{
    const int hgroups = (D.heads + HPW - 1) / HPW, tiles = (D.n + 15) / 16;
    int waves = 4, qtiles = 1;
    if (HPW == 1) {
        const TileSplit split = split_tiles(tiles, 3);
        qtiles = split.groups;
        waves = split.each;
    } else {
        const int qt = f32::AttnShape<DP, HPW>::QT;
        qtiles = (D.n + qt - 1) / qt;
    }
    const long blocks = ((long)D.B * D.R * hgroups * qtiles + 7) / 8 * 8;
    if (blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((f32::k_attention<DP, HPW, VEC>), dim3((unsigned)blocks), dim3(64 * waves), 0, st, qkv, Ir, o, D, hgroups,
                       qtiles, attention_by_image(D, hgroups), adds, nullptr, nullptr);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

// Heads side by side in a workgroup where a region's tokens do not fill four 16-row tiles.
int heads_per_group(const Dims &D)
{
    const int want = D.n <= 16 ? 4 : (D.n <= 32 ? 2 : 1);
    return D.heads > want / 2 ? want : (D.heads >= 2 ? 2 : 1);
}

// adds: to what o holds (LCE(V)).
int launch_attention(const Dims &D, const float *qkv, const int32_t *Ir, float *o, bool adds, hipStream_t st)
{
    ProfScope ps(st, K_GEN_ATTENTION);
    if (D.d > kAttnF32MaxD) {
        hipLaunchKernelGGL(gen_attention, dim3(D.B * D.R * D.heads), dim3(256), D.k * sizeof(int), st, qkv, Ir, o, D,
                           D.scale, adds);
        return launched() ? BRA_OK : BRA_ERR_LAUNCH;
    }
    const int hpw = heads_per_group(D);
    const bool vec = D.d % 4 == 0;
    if (D.d <= 32) {
        if (hpw == 4) return vec ? launch_attention_t<32, 4, true>(D, qkv, Ir, o, adds, st) : launch_attention_t<32, 4, false>(D, qkv, Ir, o, adds, st);
        if (hpw == 2) return vec ? launch_attention_t<32, 2, true>(D, qkv, Ir, o, adds, st) : launch_attention_t<32, 2, false>(D, qkv, Ir, o, adds, st);
        return vec ? launch_attention_t<32, 1, true>(D, qkv, Ir, o, adds, st) : launch_attention_t<32, 1, false>(D, qkv, Ir, o, adds, st);
    }
    if (hpw >= 2) return vec ? launch_attention_t<64, 2, true>(D, qkv, Ir, o, adds, st) : launch_attention_t<64, 2, false>(D, qkv, Ir, o, adds, st);
    return vec ? launch_attention_t<64, 1, true>(D, qkv, Ir, o, adds, st) : launch_attention_t<64, 1, false>(D, qkv, Ir, o, adds, st);
}

// Query tiles of k_attention_out: as in k_attention, in fours also where eights would leave compute units without any.
TileSplit out_split(const Dims &D)
{
    const int tiles = (D.n + 15) / 16;
    const TileSplit split = tiles <= 2 ? TileSplit{2, 1} : split_tiles(tiles, 4);
    return split.each > 4 && (long)D.B * D.R * split.groups < 256 ? TileSplit{4, (tiles + 3) / 4} : split;
}

// Attention and Y = O Wo in one kernel: two or four heads of 32 channels.  For two that is a launch and two passes over O less, 2 us on 3000 tokens and 9 on
// 50000 (16 x 56 x 56 x 64, k = 1: 61.7 -> 57.2; 60 x 28 x 28, k = 1 69.5 -> 63.8; 2 x 112 x 112, S = 16, k = 4 59.2 -> 54.3; 2 x 80 x 80, S = 8 54.1 -> 49.5);
// but both heads share a compute unit, and a block of keys takes its wavefronts' time, a microsecond for four: longer than the apart ones by blocks *
// (together - apart).  More than three times as long they stay apart, and beyond two rounds of workgroups where it is more than the apart time itself,
// counting the wavefronts that have queries.  Together / apart, us, by that ratio: 1.0: 6 x 84 x 56, k = 2 0.96 of the time; 1.7: 6 x 112 x 32, S = 8, k = 5 1.02;
// 2.0: 2 x 98 x 84, k = 2 64.2 / 62.1; 2.3: 6 x 56 x 56, S = 8, k = 8 66.5 / 63.5, 3 x 70 x 70, k = 4 67.4 / 63.2; 3.0: 2 x 84 x 84, k = 4 77.2 / 70.6; against that in fewer
// rounds 2.0: 1 x 84 x 70, k = 1 0.95; 1 x 56 x 56, k = 2, 3 and 8 24.2, 27.7, 42.0 / 25.4, 27.6, 36.8; 2 x 64 x 64, S = 4, k = 4 73.2 / 61.7.  Left on the wrong side: 13 x
// 42 x 56, k = 3 (three tiles in four wavefronts, 0.6) 60.0 / 58.0.  Apart for the shortest maps (1 x 40 x 40, S = 4, k = 2 32.7 / 31.9) and many keys
// (1 x 128 x 128, S = 8, k = 4, 16 blocks 79.6 / 82.5; S = 4, 64 blocks 236.9 / 233.6).
// Four heads of 32, in regions of at most 16 tokens, share a workgroup anyway: 6 x 28 x 28 x 128, k = 4 35.8 -> 32.1 us, 40 images 92.6 -> 88.0, 1 x
// 14 x 14 25.0 -> 20.3, 24 x 21 x 21 56.1 -> 53.6; but each region reads all of Wo and multiplies a tile of 16 rows: 64 x 14 x 14 x 128 (3136 regions of
// 4 tokens), k = 16 76.8 and 83.1.
bool attention_with_out(const Dims &D)
{
    if (D.C == 128 && D.d == 32 && D.n <= 16) return D.n > 9 || (long)D.B * D.R <= 1200;
    if (D.C != 64 || D.d != 32 || (long)D.B * D.N < 2048) return false;
    const int tiles = (D.n + 15) / 16;
    const TileSplit one = split_tiles(tiles, 3), both = out_split(D);
    const long regions = (long)D.B * D.R, blocks = (D.kn + 63) / 64;
    const long apart = tiles <= 2 ? (regions + 255) / 256 * 4 : (regions * 2 * one.groups + 255) / 256 * one.each;
    const long together = (regions * both.groups + 255) / 256 * 2 * both.each;
    const long busy = together / both.each * std::min(both.each, tiles);
    return blocks <= 32 && blocks * (together - apart) <= 3 * apart && (apart <= 10 || blocks * (busy - apart) <= apart);
}

// o holds LCE(V).
int launch_attention_out(const Dims &D, const float *qkv, const int32_t *Ir, const float *o, const float *Wo, float *Y, hipStream_t st)
{
    const TileSplit split = D.C == 128 ? TileSplit{2, 1} : out_split(D);
    const long blocks = ((long)D.B * D.R * split.groups + 7) / 8 * 8;
    if (blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, K_GEN_ATTENTION);
    const dim3 grid((unsigned)blocks), threads(128 * split.each);
    if (D.C == 128) {
        hipLaunchKernelGGL((f32::k_attention<32, 4, true, true>), grid, threads, 0, st, qkv, Ir, const_cast<float *>(o), D, 1, 1, attention_by_image(D, 1), true, Wo, Y);
        return launched() ? BRA_OK : BRA_ERR_LAUNCH;
    }
    const size_t smem = f32::out_lds_bytes(split.each);
    if (split.each == 2) hipLaunchKernelGGL(f32::k_attention_out<4>, grid, threads, smem, st, qkv, Ir, o, Wo, Y, D, split.groups);
    else hipLaunchKernelGGL(f32::k_attention_out<2>, grid, threads, smem, st, qkv, Ir, o, Wo, Y, D, split.groups);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

template <typename T>
int forward_t(const Dims &D, const T *X, const T *Wqkv, const T *Wo, const T *Wlce, T *Y,
              int32_t *Ir_out_opt, const int32_t *Ir_in_opt, void *ws, hipStream_t st)
{
    GenericWs w = carve(D, ws);
    if constexpr (std::is_same<T, float>::value) {
        if (f32_small_ok(D))
            return f32_small_forward(D, X, Wqkv, Wo, Wlce, Y, Ir_out_opt, Ir_in_opt, w.qkv, w.qk, w.qk + (size_t)D.B * D.R * D.C, st);
    }
    const long M = (long)D.B * D.N;
    const int C = D.C;
    const f32::GemmJob<T, T, float> qkv_job = {X, Wqkv, w.qkv, M, C, 3 * C, 3 * C, 3 * C, C, nullptr, nullptr, 0};
    const int32_t *Ir = Ir_in_opt;
    bool adds = false;
    int rc;
    if (!Ir_in_opt) {
        int32_t *dst = Ir_out_opt ? Ir_out_opt : w.ir;
        if (means_from_projection(D)) {
            ProfScope ps(st, K_GEN_GEMM_QKV);
            rc = launch_gemm_means<T>(D, X, Wqkv, w.qkv, w, st);
        } else {
            launch_pool<T>(D, X, w.xr, st);
            const f32::GemmJob<float, T, float> rj = region_job<T>(D, Wqkv, w);
            ProfScope ps(st, K_GEN_GEMM_QKV);
            rc = launch_gemm<false>(qkv_job, &rj, st);
        }
        if (rc != BRA_OK) return rc;
        // LCE(V) into the output map beside the routing; the attention adds itself to it
        rc = launch_route_lce(D, w, lce::Taps(Wlce), dst, adds, st);
        if (rc != BRA_OK) return rc;
        Ir = dst;
    } else {
        if (Ir_out_opt && hipMemcpyAsync(Ir_out_opt, Ir_in_opt, sizeof(int32_t) * (size_t)D.B * D.R * D.k,
                                         hipMemcpyDeviceToDevice, st) != hipSuccess)
            return BRA_ERR_LAUNCH;
        ProfScope ps(st, K_GEN_GEMM_QKV);
        rc = launch_gemm<false>(qkv_job, (const f32::GemmJob<float, T, float> *)nullptr, st);
        if (rc != BRA_OK) return rc;
    }
    if constexpr (std::is_same<T, float>::value) {
        if (adds && attention_with_out(D)) return launch_attention_out(D, w.qkv, Ir, w.o, Wo, Y, st);
    }
    rc = launch_attention(D, w.qkv, Ir, w.o, adds, st);
    if (rc != BRA_OK) return rc;
    if (!adds) {
        rc = lce::launch_lce<float>(D, w.qkv + 2 * C, 3 * C, lce::Taps(Wlce), w.o, C, K_GEN_LCE, st);
        if (rc != BRA_OK) return rc;
    }
    ProfScope ps(st, K_GEN_GEMM_WO);
    return launch_gemm<false>(f32::GemmJob<float, T, T>{w.o, Wo, Y, M, C, C, C, C, C, nullptr, nullptr, 0},
                              (const f32::GemmJob<float, T, float> *)nullptr, st);
}

// ---------------------------------------------------------------------------
// Whole block (Sec. 3.4) with scalar kernels.  One wavefront per token; lane l owns channels
// l, l + 64, ..  POS: Sum = A + DWConv3x3(A) + bpos (cross-correlation, zero padding 1);
// otherwise Sum = A + Badd.  Norm = LayerNorm(Sum) over the token's C channels from the
// float32 values (biased variance, eps inside the root), which wait in LDS between the passes.
template <typename T, bool POS>
__global__ __launch_bounds__(256) void gen_token_ln(const T *A, const T *__restrict__ Badd, const T *__restrict__ Wpos,
                                                    const float *__restrict__ bpos, const float *__restrict__ gamma,
                                                    const float *__restrict__ beta, T *Sum, T *__restrict__ Norm,
                                                    int H, int W, int C, long tokens, float eps)
{
    extern __shared__ float strips[];                 // [4 wavefronts][C]
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    float *strip = strips + (size_t)wave * C;
    const long tok = (long)blockIdx.x * 4 + wave;
    if (tok >= tokens) return;                        // whole wavefronts leave; no barrier follows
    const int x = (int)(tok % W), y = (int)((tok / W) % H);
    const T *centre = A + (size_t)tok * C;
    float s = 0.f;
    for (int c = lane; c < C; c += kWave) {
        float v = load_f32(centre + c);
        if (POS) {
            float acc = v + bpos[c];
            for (int ky = 0; ky < 3; ++ky) {
                const int yy = y + ky - 1;
                if (yy < 0 || yy >= H) continue;
                for (int kx = 0; kx < 3; ++kx) {
                    const int xx = x + kx - 1;
                    if (xx < 0 || xx >= W) continue;
                    acc = fmaf(load_f32(Wpos + (size_t)c * 9 + 3 * ky + kx),
                               load_f32(centre + ((long)(ky - 1) * W + (kx - 1)) * C + c), acc);
                }
            }
            v = acc;
        } else {
            v += load_f32(Badd + (size_t)tok * C + c);
        }
        strip[c] = v;
        s += v;
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    const float mean = s / (float)C;
    float q = 0.f;
    for (int c = lane; c < C; c += kWave) { const float d = strip[c] - mean; q = fmaf(d, d, q); }
    for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off);
    const float rstd = 1.0f / sqrtf(q / (float)C + eps);
    for (int c = lane; c < C; c += kWave) {
        const float v = strip[c];
        store_from_f32(Sum + (size_t)tok * C + c, v);             // may overwrite A: this lane has read it
        store_from_f32(Norm + (size_t)tok * C + c, fmaf((v - mean) * rstd, gamma[c], beta[c]));
    }
}

// The same where C is a multiple of 4: L lanes (a power of two) share a token, a lane has NC times 4 neighbouring channels, L apart, with their
// taps in registers for the group's `per` tokens; all that a token needs is requested before any of it is used.  One channel per
// lane and step, its nine neighbours and taps loaded one after the other behind a branch each, took 23.2 us at 392 tokens of 512 channels, now 6.2,
// and 43.6 at 31360 tokens of 96 in bf16, now 18.5 (without the position 13.8, now 8.8).
template <typename T, bool POS, int NC>
__global__ __launch_bounds__(256) void gen_token_ln4(const T *A, const T *__restrict__ Badd, const T *__restrict__ Wpos,
                                                     const float *__restrict__ bpos, const float *__restrict__ gamma,
                                                     const float *__restrict__ beta, T *Sum, T *__restrict__ Norm,
                                                     int H, int W, int C, long tokens, float eps, int L, int per)
{
    const int l = threadIdx.x % L;
    const long first = ((long)blockIdx.x * (256 / L) + threadIdx.x / L) * per;
    int c[NC];
    bool has[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        has[u] = 4 * (l + L * u) < C;
        c[u] = has[u] ? 4 * (l + L * u) : 0;
    }
    mfma::f32x4 taps[POS ? NC : 1][9], bias[POS ? NC : 1], ga[NC], be[NC];       // taps: 9 of each of the 4 channels, as they lie
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        ga[u] = *(const mfma::f32x4 *)(gamma + c[u]);
        be[u] = *(const mfma::f32x4 *)(beta + c[u]);
        if (POS) {
            bias[u] = *(const mfma::f32x4 *)(bpos + c[u]);
#pragma unroll
            for (int e = 0; e < 9; ++e) taps[u][e] = f32::load4<true>(Wpos + (size_t)c[u] * 9 + 4 * e, 4);
        }
    }
    for (long tok = first; tok < first + per; ++tok) {
        const bool valid = tok < tokens;           // the lanes of a wavefront stay together
        const long at = valid ? tok : tokens - 1;
        const int x = (int)(at % W), y = (int)((at / W) % H);
        const T *centre = A + (size_t)at * C;
        mfma::f32x4 v[NC], near[POS ? NC : 1][9];
        bool in[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) in[t] = (unsigned)(y + t / 3 - 1) < (unsigned)H && (unsigned)(x + t % 3 - 1) < (unsigned)W;
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            if (POS) {
#pragma unroll
                for (int t = 0; t < 9; ++t) near[u][t] = f32::load4<true>(centre + (in[t] ? (long)(t / 3 - 1) * W + t % 3 - 1 : 0) * C + c[u], 4);
            } else {
                v[u] = f32::load4<true>(centre + c[u], 4) + f32::load4<true>(Badd + (size_t)at * C + c[u], 4);
            }
        }
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            if (POS) {
                v[u] = near[u][4] + bias[u];
#pragma unroll
                for (int t = 0; t < 9; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int e = 9 * j + t;
                        v[u][j] = in[t] ? fmaf(taps[u][e / 4][e % 4], near[u][t][j], v[u][j]) : v[u][j];
                    }
            }
            if (has[u]) s += (v[u][0] + v[u][1]) + (v[u][2] + v[u][3]);
        }
        for (int off = L / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
        const float mean = s / (float)C;
        float q = 0.f;
#pragma unroll
        for (int u = 0; u < NC; ++u)
            if (has[u])
#pragma unroll
                for (int j = 0; j < 4; ++j) { const float d = v[u][j] - mean; q = fmaf(d, d, q); }
        for (int off = L / 2; off > 0; off >>= 1) q += __shfl_xor(q, off);
        const float rstd = 1.0f / sqrtf(q / (float)C + eps);
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            if (!valid || !has[u]) continue;
            mfma::f32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = fmaf((v[u][j] - mean) * rstd, ga[u][j], be[u][j]);
            f32::store4<true>(Sum + (size_t)tok * C + c[u], v[u], 4);     // may overwrite A: this lane has read it
            f32::store4<true>(Norm + (size_t)tok * C + c[u], o, 4);
        }
    }
}

// Tokens per group of lanes: one each up to eight workgroups per compute unit, then as many as keep them (block of 64 x 28 x 28 x 96, bf16: 159.8 us, at
// four workgroups per unit 164.6, at sixteen 159.9).
template <typename T, bool POS>
void launch_token_ln(const Dims &D, const T *A, const T *Badd, const T *Wpos, const float *bpos, const float *gamma, const float *beta, T *Sum, T *Norm,
                     float eps, hipStream_t st)
{
    const long M = (long)D.B * D.N;
    int L = 1;
    while (L < kWave && 4 * L < D.C) L *= 2;
    const int nc = (D.C + 4 * L - 1) / (4 * L);
    if (D.C % 4 == 0 && nc <= 4) {
        const long groups = 256 / L, per = std::max<long>(1, M / (groups * 2048));
        const dim3 grid((unsigned)((M + groups * per - 1) / (groups * per)));
        auto go = [&](auto n) {
            hipLaunchKernelGGL((gen_token_ln4<T, POS, decltype(n)::value>), grid, dim3(256), 0, st, A, Badd, Wpos, bpos, gamma, beta, Sum, Norm, D.H, D.W, D.C, M,
                               eps, L, (int)per);
        };
        if (nc == 1) go(std::integral_constant<int, 1>{});
        else if (nc == 2) go(std::integral_constant<int, 2>{});
        else if (nc == 3) go(std::integral_constant<int, 3>{});
        else go(std::integral_constant<int, 4>{});
        return;
    }
    hipLaunchKernelGGL((gen_token_ln<T, POS>), dim3((unsigned)((M + 3) / 4)), dim3(256), (size_t)4 * D.C * sizeof(float), st, A, Badd, Wpos, bpos, gamma, beta,
                       Sum, Norm, D.H, D.W, D.C, M, eps);
}

struct GenBlockWs {
    void *x1, *xn, *y, *hd, *inner;
    size_t bytes;
};

GenBlockWs carve_gen_block(const Dims &D, int hidden, size_t bra_bytes, void *ws)
{
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void *ptr = base ? base + off : nullptr;
        off += align256(bytes);
        return ptr;
    };
    const size_t es = D.dtype == BRA_BF16 ? 2 : 4, tokens = (size_t)D.B * D.N;
    GenBlockWs w;
    w.x1 = take(tokens * D.C * es);
    w.xn = take(tokens * D.C * es);
    w.y = take(tokens * D.C * es);
    w.hd = take(tokens * hidden * es);
    w.inner = take(bra_bytes);
    w.bytes = off;
    return w;
}

template <typename T>
int block_t(const Dims &D, int hidden, float eps, const T *X, const bra_block_params &p, T *Xout, int32_t *Ir_out_opt,
            const int32_t *Ir_in_opt, void *ws, size_t bra_bytes, int path, hipStream_t st)
{
    const GenBlockWs w = carve_gen_block(D, hidden, bra_bytes, ws);
    T *x1 = (T *)w.x1, *xn = (T *)w.xn, *y = (T *)w.y, *hd = (T *)w.hd;
    const long M = (long)D.B * D.N;
    {
        ProfScope ps(st, K_BLK_POS_LN);
        launch_token_ln<T, true>(D, X, nullptr, (const T *)p.Wpos, p.bpos, p.ln1_gamma, p.ln1_beta, x1, xn, eps, st);
    }
    if (hipGetLastError() != hipSuccess) return BRA_ERR_LAUNCH;
    int rc = (path == BRA_PATH_MFMA)
                 ? mfma_forward(D, xn, p.Wqkv, p.Wo, p.Wlce, y, Ir_out_opt, Ir_in_opt, w.inner, st)
                 : generic_forward(D, xn, p.Wqkv, p.Wo, p.Wlce, y, Ir_out_opt, Ir_in_opt, w.inner, st);
    if (rc != BRA_OK) return rc;
    {
        ProfScope ps(st, K_BLK_ADD_LN);
        launch_token_ln<T, false>(D, x1, y, nullptr, nullptr, p.ln2_gamma, p.ln2_beta, x1, xn, eps, st);
    }
    const f32::GemmJob<float, T, float> *none = nullptr;
    {
        ProfScope ps(st, K_BLK_MLP_IN);
        rc = launch_gemm<false>(f32::GemmJob<T, T, T>{xn, (const T *)p.W1, hd, M, D.C, hidden, hidden, hidden, D.C, p.b1,
                                                      nullptr, 1}, none, st);
        if (rc != BRA_OK) return rc;
    }
    ProfScope ps(st, K_BLK_MLP_OUT);
    return launch_gemm<false>(f32::GemmJob<T, T, T>{hd, (const T *)p.W2, Xout, M, hidden, D.C, D.C, D.C, hidden, p.b2, x1, 0},
                              none, st);
}

// ---------------------------------------------------------------------------
// Backward pass with fixed routing (the top-k of Eq. 5 has no derivative) in float32.
// With dO = dY Wo^T and, per query token t of region i and head h, P = softmax over the keys G_i:
//   dP_j = dO_h[t] . V_h[j],  dS_j = P_j (dP_j - sum_u P_u dP_u),
//   dQ_h[t] = scale sum_j dS_j K_h[j],  dK_h[j] += scale dS_j Q_h[t],  dV_h[j] += P_j dO_h[t].
// The weight gradients come from per-workgroup partial sums, added in a fixed order.
constexpr int kBwdMaxD = kAttnF32MaxD;

// Token shares of the weight-gradient contractions: about 1024 workgroups over the 64 x 64 output blocks of
// both products.
struct SharePlan {
    int shares, tokens;
};

SharePlan share_plan(long M, int C)
{
    const long blocks = (long)((C + 63) / 64) * ((3 * C + 63) / 64 + (C + 63) / 64), steps = (M + 31) / 32;
    const long want = 1024 / blocks > 1 ? 1024 / blocks : 1, per = (steps + want - 1) / want;
    return {(int)((steps + per - 1) / per), (int)(per * 32)};
}

// Which gradients k_heads_bwd_q and k_heads_bwd_kv take.  Channels per thread of the passes: those of the attention kernels that carry them (one with
// these, else two with 4-channel loads).  Two workgroups
// per compute unit (29 x 28 x 28 x 96: whole gradient 176 us, 182 with three).
bool by_heads(const Dims &D) { return D.n <= 32 && D.d <= 32; }

// The query side of regions of 17 to 32 tokens that keeps all keys as one block of 64 instead of in tiles of 16 by wavefront: with two tiles of queries a wavefront of
// k_heads_bwd_q keeps two tiles of keys.  Whole gradient (us), it / the block: 6 x 35 x 35 x 192, k = 2 154 / 140, 8 images 183 / 173, 2 images 74.0 / 68.1; 12 x 35 x 35 x 96 bf16, k = 2
// 119 / 112; 24 x 21 x 42 x 64, k = 3 116 / 107; the other way round 7 x 21 x 42 x 64, k = 2 53.3 / 55.9; with more keys 10 x 35 x 35 x 96, k = 3 123 / 140; with one block of 32
// mixed, 10 x 35 x 35 x 96, k = 1 99.6 / 105.0, 2 x 35 x 35 x 192 68.4 / 66.2, 14 x 28 x 56 x 64 90.5 / 87.3.
bool query_by_heads(const Dims &D) { return by_heads(D) && !(D.n > 16 && D.heads >= 2 && D.kn > 32 && D.kn <= 64); }
lce::LcePlan lce_grad_plan(const Dims &D) { return lce::lce_plan(D, 512, D.d % 4 == 0 && !query_by_heads(D) ? 8 : 4); }

struct BwdWs {
    float *qkv, *o, *dO, *dqkv, *lse, *dsum, *part_qkv, *part_o, *part_lce;
    size_t bytes;
};

BwdWs carve_bwd(const Dims &D, void *ws)
{
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t count) {
        void *ptr = base ? base + off : nullptr;
        off += align256(count * sizeof(float));
        return (float *)ptr;
    };
    const size_t tok = (size_t)D.B * D.N, C = D.C;
    const int shares = share_plan((long)tok, D.C).shares;
    BwdWs w;
    w.qkv = take(tok * 3 * C);
    w.o = take(tok * C);
    w.dO = take(tok * C);
    w.dqkv = take(tok * 3 * C);
    w.lse = take(tok * D.heads);
    w.dsum = take(tok * D.heads);
    w.part_qkv = take((size_t)shares * 3 * C * C);
    w.part_o = take((size_t)shares * C * C);
    w.part_lce = take((size_t)lce_grad_plan(D).groups * 25 * C);
    w.bytes = off;
    return w;
}

// The query side, or both, by workgroups of HPW heads.
template <int DP, int HPW, bool VEC, bool KEYS = true>
int launch_attn_bwd_t(const Dims &D, const BwdWs &w, const int32_t *Ir, const lce::Taps &taps, hipStream_t st)
{
    const int hgroups = (D.heads + HPW - 1) / HPW, qt = f32::AttnShape<DP, HPW>::QT, tiles = (D.n + qt - 1) / qt;
    const long blocks = ((long)D.B * D.R * hgroups * tiles + 7) / 8 * 8;
    const bool by_image = gradients_by_image(D, hgroups, blocks);
    // The passes of the depth-wise convolution's gradients lie behind the workgroups of the attention: the one with the tap
    // gradients beside the query side, which leaves dV to be added to by the key side, O += LCE(V) beside the key side.  In
    // front of the query side it was slower (4 x 56 x 56 x 64, k = 2: 100.9 us behind, 105.6 in front).
    const float *V = w.qkv + 2 * D.C;
    const lce::GradJob<float> grad = {w.dO, V, taps, w.dqkv + 2 * D.C, w.part_lce, 3 * D.C, 3 * D.C, lce_grad_plan(D)};
    const lce::AddJob<float> add = KEYS ? lce::add_job<float>(D, V, 3 * D.C, taps, w.o, D.C, VEC ? 2 : 1, 256) : lce::AddJob<float>{};
    if (blocks + std::max(grad.p.blocks(), add.blocks) > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((f32::k_attn_bwd_q<DP, HPW, VEC>), dim3((unsigned)(blocks + grad.p.blocks())), dim3(256), 0, st, w.qkv, w.dO, Ir, w.o, w.dqkv, w.lse,
                       w.dsum, D, hgroups, tiles, by_image, grad, grad.p.blocks());
    if constexpr (!KEYS) return launched() ? BRA_OK : BRA_ERR_LAUNCH;
    else hipLaunchKernelGGL((f32::k_attn_bwd_kv<DP, HPW, VEC>), dim3((unsigned)(blocks + add.blocks)), dim3(256), 0, st, w.qkv, w.dO, Ir, w.lse,
                       w.dsum, w.dqkv, D, hgroups, tiles, by_image, add, add.blocks);
    if (!launched()) return BRA_ERR_LAUNCH;
    return add.blocks ? BRA_OK : lce::launch_lce<float>(D, V, 3 * D.C, taps, w.o, D.C, K_GEN_BACKWARD, st);
}

// Wavefronts that share a head of a region: a chain of rows is hidden by the other wavefronts of the unit or by more of them on it, and each reads the region's own rows.
// us, query side / key side with 1, 2, 4 per head: 588 heads of regions (4 x 14 x 28 x 96, k = 16) 18.1, 15.7, 13.8 / 16.5, 14.1, 11.5; 1568 (8 x 28 x 28 x 128, k = 4)
// 18.1, 22.0, 25.4 / 21.1, 16.8, 20.8; 3072 (3 x 32 x 32 x 128, S = 16, k = 11) 19.9, 23.3, 28.6 / 24.2, 29.6, 41.4.
// A workgroup has four wavefronts: at least as many per head as leave none without one.
int least_share(const Dims &D) { return D.heads >= 3 ? 1 : D.heads == 2 ? 2 : 4; }

// Query side: no more than it has tiles of 16 routed keys.  Whole gradient of B x 28 x 28 x 128, us, 4, 2, 1: k = 4, 588 heads of regions 52.9, 53.1, 54.0; 784 58.5, 55.6, 56.8; 980 64.6, 61.5,
// 61.4; 1176 70.7, 69.3, 69.0; 1372 74.9, 70.7, 71.0; 1568 79.3, 77.4, 74.5.  But as many as keep all weights in registers (kKeptTiles): k = 8 (8 tiles) 1372 84.6, 79.8, 87.0; 2744 134.7, 131.4, 132.1; k = 16
// (16) 1372 102.0, 103.8, 114.9; 2744 167.8, 177.3, 175.6.  With two tiles of queries, which keep half, two up to 3200, where four heads at a time leave places empty or
// there are many tiles: 8 x 35 x 35 x 192, k = 3 187, 184, 197, k = 5 205, 207, 234, k = 8
// 254, 245, 289; 16 x 35 x 35 x 96, k = 3 174, 178, 180, k = 8 243, 257, 270; 8 x 28 x 56 x 192, k = 8 297, 296, 353; 12 x 35 x 35 x 128, k = 3 -, 164, 163, k = 5 -, 184, 198; 24 x 35 x 35 x 96, k = 4 (3528) -, 238, 230.
int query_share(const Dims &D)
{
    const long heads = (long)D.B * D.R * D.heads;
    const int tiles = (D.kn + 15) / 16, keeps = D.n > 16 ? (heads <= 3200 && tiles > (D.heads % 4 ? 2 : 5) ? 2 : 1) : tiles <= 4 || tiles > 16 ? 1 : tiles <= 8 ? 2 : 4;
    const int share = std::max(keeps, heads <= 600 ? 4 : heads <= 1200 ? 2 : 1);
    return std::max(least_share(D), std::min(share, tiles >= 4 ? 4 : tiles >= 2 ? 2 : 1));
}

// Key side: no more than the rows of an average list are worth, which has k n.  Whole gradient, us, 4, 2, 1: 784 heads of regions, 2 x 14 x 14 x 256, k = 1 (4 rows) 50.6, 46.8, 46.1; 4 x 14 x 28 x 128,
// k = 2 (16) 45.9, 45.3, 45.1; 4 x 28 x 28 x 128, k = 2 (32) 53.6, 52.5, 54.8, k = 4 (64) 55.6, 54.9, 58.7, k = 8 62.7, 62.9, 68.4, k = 16 79.1, 81.0, 88.0; 588, k = 4 52.9, 53.4, 56.4.  One or two,
// 64 rows: 1372 -, 70.8, 73.8; 1568 -, 74.5, 76.6; 1764 -, 82.9, 83.5; 2352 -, 102.6, 102.9; 2744 -, 109.1, 107.5; 4 tokens a region and 64 rows 1568 -, 64.8, 64.2, 1960 -, 69.9, 67.5.
// With two tiles of keys, from 32 rows on, two up to twice as many: 8 x 35 x 35 x 192, k = 2 (2352) -, 170, 173, k = 5 211, 207, 228; 24 x 35 x 35 x 96, k = 2 (3528) 188, 184, 181.  And a row is worth more: 7 x 35 x 35 x 64, k = 2 (50) 60.7, 64.1, -, k = 1 57.8, 59.1, -; 2 x 35 x 35 x 192, k = 1 68.0, 69.0, -; 5 x 21 x 42 x 96, k = 1 (18) 61.8, 59.5, 58.7.
int key_share(const Dims &D)
{
    const long heads = (long)D.B * D.R * D.heads;
    const int share = heads <= 800 ? 4 : heads <= (D.n > 16 && D.kn >= 32 ? 3200 : 1600) ? 2 : 1, rows = D.n > 16 ? 3 * D.kn : D.kn;
    return std::max(least_share(D), std::min(share, rows >= 64 ? 4 : rows >= 16 ? 2 : 1));
}

template <int NT, bool VEC>
int launch_heads_bwd(const Dims &D, const BwdWs &w, const int32_t *Ir, const lce::Taps &taps, hipStream_t st)
{
    const float *V = w.qkv + 2 * D.C;
    const lce::GradJob<float> grad = {w.dO, V, taps, w.dqkv + 2 * D.C, w.part_lce, 3 * D.C, 3 * D.C, lce_grad_plan(D)};
    const lce::AddJob<float> add = lce::add_job<float>(D, V, 3 * D.C, taps, w.o, D.C, VEC ? 2 : 1, 256);
    // workgroups of a side with `share` wavefronts per head
    auto groups = [&](int share) { return (D.heads + 4 / share - 1) / (4 / share); };
    auto blocks = [&](int share) { return ((long)D.B * D.R * groups(share) + 7) / 8 * 8; };
    const int of_query = query_share(D), of_key = key_share(D);
    if (blocks(std::max(of_query, of_key)) + std::max(grad.p.blocks(), add.blocks) > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    auto query_side = [&](auto share) {
        constexpr int W = decltype(share)::value;
        hipLaunchKernelGGL((f32::k_heads_bwd_q<NT, W, VEC>), dim3((unsigned)(blocks(W) + grad.p.blocks())), dim3(256), 0, st, w.qkv, w.dO, Ir, w.o, w.dqkv,
                           w.lse, w.dsum, D, groups(W), gradients_by_image(D, groups(W), blocks(W)), grad, grad.p.blocks());
    };
    auto key_side = [&](auto share) {
        constexpr int W = decltype(share)::value;
        hipLaunchKernelGGL((f32::k_heads_bwd_kv<NT, W, VEC>), dim3((unsigned)(blocks(W) + add.blocks)), dim3(256), 0, st, w.qkv, w.dO, Ir, w.lse, w.dsum,
                           w.dqkv, D, groups(W), gradients_by_image(D, groups(W), blocks(W)), add, add.blocks);
    };
    auto launch = [&](int share, auto side) {
        if (share == 4) side(std::integral_constant<int, 4>{});
        else if (share == 2) side(std::integral_constant<int, 2>{});
        else side(std::integral_constant<int, 1>{});
    };
    bool apart = false;
    if constexpr (NT == 2) {
        apart = !query_by_heads(D);
        if (apart) {
            const int rc = launch_attn_bwd_t<32, 2, VEC, false>(D, w, Ir, taps, st);
            if (rc != BRA_OK) return rc;
        }
    }
    if (!apart) launch(of_query, query_side);
    launch(of_key, key_side);
    if (!launched()) return BRA_ERR_LAUNCH;
    return add.blocks ? BRA_OK : lce::launch_lce<float>(D, V, 3 * D.C, taps, w.o, D.C, K_GEN_BACKWARD, st);
}

int launch_attn_bwd(const Dims &D, const BwdWs &w, const int32_t *Ir, const lce::Taps &taps, hipStream_t st)
{
    const bool vec = D.d % 4 == 0;
    if (by_heads(D)) {
        if (D.n <= 16) return vec ? launch_heads_bwd<1, true>(D, w, Ir, taps, st) : launch_heads_bwd<1, false>(D, w, Ir, taps, st);
        return vec ? launch_heads_bwd<2, true>(D, w, Ir, taps, st) : launch_heads_bwd<2, false>(D, w, Ir, taps, st);
    }
    if (D.d <= 32) return vec ? launch_attn_bwd_t<32, 1, true>(D, w, Ir, taps, st) : launch_attn_bwd_t<32, 1, false>(D, w, Ir, taps, st);
    if (heads_per_group(D) >= 2) return vec ? launch_attn_bwd_t<64, 2, true>(D, w, Ir, taps, st) : launch_attn_bwd_t<64, 2, false>(D, w, Ir, taps, st);
    return vec ? launch_attn_bwd_t<64, 1, true>(D, w, Ir, taps, st) : launch_attn_bwd_t<64, 1, false>(D, w, Ir, taps, st);
}

// The gradients take five launches: the products of the recomputation, query side and key side (each with a depth-wise pass),
// the products that end them, the sums of the partial matrices.  With a launch for each of the eight kernels (us): 8 x 28 x 28
// x 128 float32, k = 4: 117 -> 91; 1 x 14 x 14 x 64: 53 -> 31; 2 x 14 x 14 x 256, k = 16: 98 -> 68; 29 x 28 x 28 x 96 bf16: 204 -> 176.
template <typename T>
int launch_gemm_both(const f32::GemmJob<T, T, float> &J0, const f32::GemmJob<T, T, float> &J1, hipStream_t st)
{
    if constexpr (std::is_same<T, float>::value) {
        if (splits(J0.M, J0.N, J0.K, J1.N)) {
            const int rows = split_rows(J0.M, J0.N, J1.N);
            const long rt = (J0.M + rows - 1) / rows, s0 = rt * (J0.N / 32), s1 = rt * (J1.N / 32);
            if (rows == 16) hipLaunchKernelGGL(f32::k_gemm_both_split<1>, dim3((unsigned)(s0 + s1)), dim3(512), 0, st, J0, J1, (int)s0);
            else hipLaunchKernelGGL(f32::k_gemm_both_split<2>, dim3((unsigned)(s0 + s1)), dim3(512), 0, st, J0, J1, (int)s0);
            return launched() ? BRA_OK : BRA_ERR_LAUNCH;
        }
    }
    const long mt = (J0.M + f32::kGemmBM - 1) / f32::kGemmBM;
    const bool narrow = J1.N <= 64 || narrow_tiles<T>(J0.M, J0.N, J1.N);
    const int bn = narrow ? 64 : 128;
    const long b0 = tile_blocks<T>(mt * ((J0.N + bn - 1) / bn)), b1 = tile_blocks<T>(mt * ((J1.N + bn - 1) / bn));
    if (b0 + b1 > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)(b0 + b1));
    const bool vec = J1.K % 4 == 0;              // all sizes and pitches are multiples of C
    if (vec && narrow) hipLaunchKernelGGL((f32::k_gemm_both<true, 64, T>), grid, dim3(256), 0, st, J0, J1, (int)b0);
    else if (vec) hipLaunchKernelGGL((f32::k_gemm_both<true, kWideBN<T>, T>), grid, dim3(256), 0, st, J0, J1, (int)b0);
    else if (narrow) hipLaunchKernelGGL((f32::k_gemm_both<false, 64, T>), grid, dim3(256), 0, st, J0, J1, (int)b0);
    else hipLaunchKernelGGL((f32::k_gemm_both<false, kWideBN<T>, T>), grid, dim3(256), 0, st, J0, J1, (int)b0);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

template <typename T>
int launch_gemm_end(const f32::TnJob<T, float> &J0, const f32::TnJob<float, T> &J1, int shares, int share_tokens, const f32::GemmJob<float, T, T> &J, hipStream_t st)
{
    const long mt = (J.M + f32::kGemmBM - 1) / f32::kGemmBM;
    const bool narrow = narrow_tiles<T>(J.M, J.N);
    const int bn = narrow ? 64 : 128;
    const long tn = ((long)(J0.blocks() + J1.blocks()) * shares + 7) / 8 * 8;
    if constexpr (std::is_same<T, float>::value) {
        // shorter contractions beside those of the weights up to 80 tiles (117 of K = 576, 2 x 35 x 35 x 192: kernel 25.0 us, 26.9 so)
        if (splits(J.M, J.N, J.K) && (J.K >= 1024 || mt * ((J.N + 63) / 64) <= 80)) {
            const dim3 grid((unsigned)(tn + (J.M + 15) / 16 * (J.N / 32)));
            hipLaunchKernelGGL((f32::k_gemm_end<true, 64, T, true>), grid, dim3(256), 0, st, J0, J1, J.M, share_tokens, (int)tn, J);
            return launched() ? BRA_OK : BRA_ERR_LAUNCH;
        }
    }
    const long blocks = tn + tile_blocks<T>(mt * ((J.N + bn - 1) / bn));
    if (blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)blocks);
    const bool vec = J.N % 4 == 0;               // all sizes and pitches are multiples of C
    if (vec && narrow) hipLaunchKernelGGL((f32::k_gemm_end<true, 64, T>), grid, dim3(256), 0, st, J0, J1, J.M, share_tokens, (int)tn, J);
    else if (vec) hipLaunchKernelGGL((f32::k_gemm_end<true, kWideBN<T>, T>), grid, dim3(256), 0, st, J0, J1, J.M, share_tokens, (int)tn, J);
    else if (narrow) hipLaunchKernelGGL((f32::k_gemm_end<false, 64, T>), grid, dim3(256), 0, st, J0, J1, J.M, share_tokens, (int)tn, J);
    else hipLaunchKernelGGL((f32::k_gemm_end<false, kWideBN<T>, T>), grid, dim3(256), 0, st, J0, J1, J.M, share_tokens, (int)tn, J);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

template <typename T>
int backward_t(const Dims &D, const T *X, const T *Wqkv, const T *Wo, const T *Wlce, const int32_t *Ir, const T *dY,
               T *dX, float *dWqkv, float *dWo, float *dWlce, void *ws, hipStream_t st)
{
    const BwdWs w = carve_bwd(D, ws);
    const long M = (long)D.B * D.N;
    const int C = D.C, C3 = 3 * D.C;
    ProfScope ps(st, K_GEN_BACKWARD);
    // forward intermediates again: Q | K | V (the attention output comes out of the query side); dO = dY Wo^T
    int rc = launch_gemm_both<T>(f32::GemmJob<T, T, float>{X, Wqkv, w.qkv, M, C, C3, C3, C3, C, nullptr, nullptr, 0},
                                 f32::GemmJob<T, T, float>{dY, Wo, w.dO, M, C, C, C, C, C, nullptr, nullptr, 0}, st);
    if (rc != BRA_OK) return rc;
    // O = attention + LCE(V) for dWo, dQ, dK, dV and the tap gradients
    rc = launch_attn_bwd(D, w, Ir, lce::Taps(Wlce), st);
    if (rc != BRA_OK) return rc;
    const lce::LcePlan lp = lce_grad_plan(D);
    // dX = [dQ | dK | dV] Wqkv^T; dWqkv = X^T [dQ | dK | dV], dWo = O^T dY
    const SharePlan sp = share_plan(M, C);
    rc = launch_gemm_end<T>(f32::TnJob<T, float>{X, w.dqkv, w.part_qkv, C, C3, C, C3},
                            f32::TnJob<float, T>{w.o, dY, w.part_o, C, C, C, C}, sp.shares, sp.tokens,
                            f32::GemmJob<float, T, T>{w.dqkv, Wqkv, dX, M, C3, C3, C, C, C3, nullptr, nullptr, 0}, st);
    if (rc != BRA_OK) return rc;
    const bwd::ReduceJob r0 = bwd::reduce_job(w.part_qkv, dWqkv, sp.shares, C3 * C), r1 = bwd::reduce_job(w.part_o, dWo, sp.shares, C * C),
                         r2 = bwd::reduce_job(w.part_lce, dWlce, lp.groups, 25 * C);
    hipLaunchKernelGGL(bwd::k_reduce_parts, dim3(r0.blocks + r1.blocks + r2.blocks), dim3(256), 0, st, r0, r1, r2);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace

int token_ln_bf16(const Dims &D, bool pos, const bf16_t *A, const bf16_t *Badd, const bra_block_params &p, const float *gamma, const float *beta, bf16_t *Sum,
                  bf16_t *Norm, float eps, hipStream_t st)
{
    if (D.C % 4 != 0 || D.C > 1024) return BRA_ERR_UNSUPPORTED;
    if (pos) launch_token_ln<bf16_t, true>(D, A, nullptr, (const bf16_t *)p.Wpos, p.bpos, gamma, beta, Sum, Norm, eps, st);
    else launch_token_ln<bf16_t, false>(D, A, Badd, nullptr, nullptr, gamma, beta, Sum, Norm, eps, st);
    return launched() ? BRA_OK : BRA_ERR_LAUNCH;
}

size_t generic_block_workspace_bytes(const Dims &D, int hidden, size_t bra_bytes)
{
    return carve_gen_block(D, hidden, bra_bytes, nullptr).bytes;
}

int generic_block_forward(const Dims &D, int hidden, float eps, const void *X, const bra_block_params &p, void *Xout,
                          int32_t *Ir_out_opt, const int32_t *Ir_in_opt, void *ws, size_t bra_bytes, int path,
                          hipStream_t st)
{
    if (D.dtype == BRA_BF16)
        return block_t<bf16_t>(D, hidden, eps, (const bf16_t *)X, p, (bf16_t *)Xout, Ir_out_opt, Ir_in_opt, ws,
                               bra_bytes, path, st);
    return block_t<float>(D, hidden, eps, (const float *)X, p, (float *)Xout, Ir_out_opt, Ir_in_opt, ws, bra_bytes,
                          path, st);
}

bool generic_backward_supported(const Dims &D)
{
    return generic_supported(D) && D.d <= kBwdMaxD && (long)D.B * D.R * D.heads * ((D.n + 15) / 16) <= 0x7fffffffL;
}

size_t generic_backward_workspace_bytes(const Dims &D) { return carve_bwd(D, nullptr).bytes; }

int generic_backward(const Dims &D, const void *X, const void *Wqkv, const void *Wo, const void *Wlce,
                     const int32_t *Ir, const void *dY, void *dX, float *dWqkv, float *dWo, float *dWlce, void *ws,
                     hipStream_t st)
{
    if (D.dtype == BRA_BF16)
        return backward_t<bf16_t>(D, (const bf16_t *)X, (const bf16_t *)Wqkv, (const bf16_t *)Wo, (const bf16_t *)Wlce,
                                  Ir, (const bf16_t *)dY, (bf16_t *)dX, dWqkv, dWo, dWlce, ws, st);
    return backward_t<float>(D, (const float *)X, (const float *)Wqkv, (const float *)Wo, (const float *)Wlce, Ir,
                             (const float *)dY, (float *)dX, dWqkv, dWo, dWlce, ws, st);
}

bool generic_supported(const Dims &D)
{
    // grid sizes must fit 31 bits; head width and region count are bounded by the
    // static buffers of the attention and top-k kernels.
    if (D.d > kAttnMaxD) return false;
    if (D.R > kMaxRegions) return false;
    if ((long)D.B * D.R * D.heads > 0x7fffffffL) return false;
    if (((long)D.B * D.N * D.C + 255) / 256 > 0x7fffffffL) return false;
    if ((size_t)D.k * sizeof(int) > 16 * 1024) return false;
    if ((size_t)D.C * sizeof(float) > 48 * 1024) return false;
    return true;
}

size_t generic_workspace_bytes(const Dims &D) { return carve(D, nullptr).bytes; }

int generic_route(const Dims &D, const void *X, const void *Wqkv, int32_t *Ir, float *Ar_opt,
                  void *ws, hipStream_t st)
{
    GenericWs w = carve(D, ws);
    if (f32_small_ok(D))      // the kernels that bra_forward runs for this shape, so that both give the same index
        return f32_small_route(D, (const float *)X, (const float *)Wqkv, Ir, Ar_opt, w.qkv, w.qk, w.qk + (size_t)D.B * D.R * D.C, st);
    if (D.dtype == BRA_F32)
        return launch_route<float>(D, (const float *)X, (const float *)Wqkv, Ir, Ar_opt, w, st);
    return launch_route<bf16_t>(D, (const bf16_t *)X, (const bf16_t *)Wqkv, Ir, Ar_opt, w, st);
}

int generic_forward(const Dims &D, const void *X, const void *Wqkv, const void *Wo,
                    const void *Wlce, void *Y, int32_t *Ir_out_opt, const int32_t *Ir_in_opt,
                    void *ws, hipStream_t st)
{
    if (D.dtype == BRA_F32)
        return forward_t<float>(D, (const float *)X, (const float *)Wqkv, (const float *)Wo,
                                (const float *)Wlce, (float *)Y, Ir_out_opt, Ir_in_opt, ws, st);
    return forward_t<bf16_t>(D, (const bf16_t *)X, (const bf16_t *)Wqkv, (const bf16_t *)Wo,
                             (const bf16_t *)Wlce, (bf16_t *)Y, Ir_out_opt, Ir_in_opt, ws, st);
}

}  // namespace bra
