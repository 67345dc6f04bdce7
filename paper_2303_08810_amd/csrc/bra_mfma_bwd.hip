// Backward pass of the layer on the matrix cores (bf16 tensors, heads of 32 or 64 channels, C a
// multiple of 64 up to 4096, at most 4096 routing entries per image), with the routing index held fixed.
//
// Chain rule through Eq. 6-7 and Eq. 1-2, with O = Attention(Q, K^g, V^g) + LCE(V), Y = O Wo:
//     dO = dY Wo^T                     beside Q, K, V, Wo taken transposed as it lies
//     P  = softmax(scale Q K^T)        recomputed per (region, head) from the re-projected Q, K
//     dP = dO V^T,  dS = scale P o (dP - D),  D = rowsum(P o dP)
//     dQ = dS K                        query side: it also leaves the row statistics (log-sum-exp and D) and the
//                                      attention output
//     dK = dS^T Q,  dV = P^T dO        key side: from the query regions routed to a KEY region, found in Ir, with P and
//                                      dS recomputed from the statistics and sums in registers: no atomic adds
//                                      (k_attn_bwd_map on small maps, else k_attn_bwd_q and k_attn_bwd_kv)
//     O += LCE(V)                      in the query side, in the key side's launch, at the end of k_attn_bwd_map, or k_lce_backward
//     dV += LCE^T(dO) (the correlation with the taps reversed; also in the key side and k_attn_bwd_map) and
//     dWlce[c][ky][kx] = sum_t dO[t][c] V[t + (ky - 2, kx - 2)][c]       in the query side's launch, k_attn_bwd_map, or k_lce_backward
//     dX = [dQ | dK | dV] Wqkv^T,  dWqkv = X^T [dQ | dK | dV]      k_bwd_proj, one pass over the gradient map, or k_gemm_bt_tn
//     dWo = O^T dY                     k_bwd_proj or k_gemm_tn (contraction over tokens)
// All products take bf16 operands and accumulate in float32; dQ, dK, dV and dO are rounded to
// bf16 between the kernels (they are matrix-core operands of the next product).  The weight
// gradients are summed from per-workgroup partial sums in a fixed order (k_reduce_parts).
#include "bra_bwd_dev.h"
#include "bra_gemm.h"
#include "bra_lce_dev.h"
#include "bra_mfma_bwd_attn.h"
#include "bra_mfma_bwd_map.h"

namespace bra {

using namespace mfma;
using bwd::k_reduce_parts;
using bwd::reduce_job;
using bwd::ReduceJob;

namespace {

template <typename K>
bool opt_in(K kernel, bool &done)
{
    if (done) return true;
    if (hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) !=
        hipSuccess)
        return false;
    done = true;
    return true;
}

// Two transposing reads -> one MFMA operand: lane 16 g + i receives column col0 + i of the
// rows row0 + 4 g .. + 3 (contraction slots 0..3) and row0 + 16 + 4 g .. + 3 (slots 4..7) of a
// row-major tile.  The same row-to-slot map on both operands of a product (or the accumulator
// layout of a preceding product as the other operand) keeps the contraction consistent.
__device__ __forceinline__ bf16x8 tr_operand(const bf16_t *T, int pitch, int row0, int col0, int g, int i)
{
    const bf16_t *p = T + (row0 + 4 * g + i / 4) * pitch + col0 + 4 * (i % 4);
    const u32x2 a0 = __builtin_bit_cast(u32x2, lds_read_tr16(p));
    const u32x2 a1 = __builtin_bit_cast(u32x2, lds_read_tr16(p + 16 * pitch));
    const u32x4 av = {a0[0], a0[1], a1[0], a1[1]};
    return __builtin_bit_cast(bf16x8, av);
}

// ---------------------------------------------------------------------------
// The two products that read the gradient map G = [dQ | dK | dV] ([M][3C]), in one pass over it:
//     dX = G Wqkv^T                    (derivative of Eq. 3 with respect to X)
//     dWqkv = X^T G                    (with respect to the weights; contraction over tokens)
// and, from the same tiles of O and dY beside them, dWo = O^T dY (Eq. 4).
// C = 64.  A group of four wavefronts streams 64-token tiles of all four maps through LDS (the next tile
// travels to registers meanwhile).  Wavefront w holds rows 16 w .. 16 w + 15 of Wqkv as A
// operands and forms dX^T[channel][token] = Wqkv G^T tile by tile (B operand: a token's row of G);
// and it keeps rows 16 w .. 16 w + 15 of dWqkv as 3C / 16 accumulators over all its tiles (both
// operands by transposing reads), written at the end as Part[workgroup][C][3C] for k_reduce_parts, and those of dWo as C / 16.
// H = 2: two such groups of wavefronts in one workgroup, tile by tile in turn, add their sums through LDS at the end:
// half as many partial matrices to write and to read again, which bound the end of the call.
struct ProjSmem {
    static constexpr int C = 64, GS = 3 * C + 8, XS = C + 8;
    static constexpr size_t bytes = (size_t)64 * (GS + 3 * XS) * 2;
};

template <int H>
__global__ __launch_bounds__(256 * H) void k_bwd_proj(const bf16_t *__restrict__ G, const bf16_t *__restrict__ X,
                                                      const bf16_t *__restrict__ Wqkv, bf16_t *__restrict__ dX,
                                                      float *__restrict__ Part, const bf16_t *__restrict__ O,
                                                      const bf16_t *__restrict__ dY, float *__restrict__ PartO, long M,
                                                      int tiles, int tiles_per_wg)
{
    constexpr int C = ProjSmem::C, NT = 4 * C, GS = ProjSmem::GS, XS = ProjSmem::XS, KS = 3 * C / 32, CT = 3 * C / 16;
    constexpr int GCH = 3 * C / 8, XCH = C / 8, GL = 64 * GCH / NT, XL = 64 * XCH / NT, OT = C / 16;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int half = H == 1 ? 0 : (int)threadIdx.x / NT, tid = threadIdx.x % NT;
    bf16_t *Gs = (bf16_t *)(smem + half * ProjSmem::bytes), *Xs = Gs + 64 * GS, *Os = Xs + 64 * XS, *Ys = Os + 64 * XS;
    const int w = tid / 64, lane = tid % 64, g = lane / 16, i = lane % 16;
    bf16x8 wf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) wf[ks] = *(const bf16x8 *)(Wqkv + (size_t)(16 * w + i) * 3 * C + 32 * ks + 8 * g);
    f32x4 acc[CT], acco[OT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ct = 0; ct < OT; ++ct) acco[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 gr[GL], xr[XL], orr[XL], yr[XL];
    auto fetch = [&](long tile) {
#pragma unroll
        for (int u = 0; u < GL; ++u) {
            const int idx = tid + NT * u;
            const size_t t = min(tile * 64 + idx / GCH, M - 1);
            gr[u] = *(const u32x4 *)(G + t * 3 * C + (idx % GCH) * 8);
        }
#pragma unroll
        for (int u = 0; u < XL; ++u) {
            const int idx = tid + NT * u;
            const size_t at = (size_t)min(tile * 64 + idx / XCH, M - 1) * C + (idx % XCH) * 8;
            xr[u] = *(const u32x4 *)(X + at);
            orr[u] = *(const u32x4 *)(O + at);
            yr[u] = *(const u32x4 *)(dY + at);
        }
    };
    const int first = blockIdx.x * tiles_per_wg, last = min(tiles, first + tiles_per_wg);
    if (first < last) fetch(first + half);
    for (int t0 = first; t0 < last; t0 += H) {
        const int tile = t0 + half;
        const long rows = H == 1 || tile < last ? M : 0;    // the second group has no tile left: it adds nothing
        if (t0 > first) __syncthreads();            // the previous tile's readers are done
        if ((long)tile * 64 + 64 > rows) {          // tokens past the end add nothing: blanked here, not behind the loads
#pragma unroll
            for (int u = 0; u < GL; ++u)
                if ((long)tile * 64 + (tid + NT * u) / GCH >= rows) gr[u] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int u = 0; u < XL; ++u)
                if ((long)tile * 64 + (tid + NT * u) / XCH >= rows) xr[u] = orr[u] = yr[u] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < GL; ++u) {
            const int idx = tid + NT * u;
            *(u32x4 *)(Gs + (idx / GCH) * GS + (idx % GCH) * 8) = gr[u];
        }
#pragma unroll
        for (int u = 0; u < XL; ++u) {
            const int idx = tid + NT * u;
            *(u32x4 *)(Xs + (idx / XCH) * XS + (idx % XCH) * 8) = xr[u];
            *(u32x4 *)(Os + (idx / XCH) * XS + (idx % XCH) * 8) = orr[u];
            *(u32x4 *)(Ys + (idx / XCH) * XS + (idx % XCH) * 8) = yr[u];
        }
        __syncthreads();
        if (t0 + H < last) fetch(tile + H);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                a = mfma16(wf[ks], *(const bf16x8 *)(Gs + (16 * rt + i) * GS + 32 * ks + 8 * g), a);
            const long t = (long)tile * 64 + 16 * rt + i;       // a[j] = dX[token t][channel 16 w + 4 g + j]
            if (t < rows) *(u32x2 *)(dX + (size_t)t * C + 16 * w + 4 * g) = pack4(a);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 xa = tr_operand(Xs, XS, 32 * ks, 16 * w, g, i);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[ct] = mfma16(xa, tr_operand(Gs, GS, 32 * ks, 16 * ct, g, i), acc[ct]);
            const bf16x8 oa = tr_operand(Os, XS, 32 * ks, 16 * w, g, i);
#pragma unroll
            for (int ct = 0; ct < OT; ++ct) acco[ct] = mfma16(oa, tr_operand(Ys, XS, 32 * ks, 16 * ct, g, i), acco[ct]);
        }
    }
    if (H == 2) {
        f32x4 *sums = (f32x4 *)smem;
        __syncthreads();
        if (half == 1) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) sums[ct * NT + tid] = acc[ct];
#pragma unroll
            for (int ct = 0; ct < OT; ++ct) sums[(CT + ct) * NT + tid] = acco[ct];
        }
        __syncthreads();
        if (half == 1) return;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] += sums[ct * NT + tid];
#pragma unroll
        for (int ct = 0; ct < OT; ++ct) acco[ct] += sums[(CT + ct) * NT + tid];
    }
    float *out = Part + (size_t)blockIdx.x * C * 3 * C;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int j = 0; j < 4; ++j) out[(size_t)(16 * w + 4 * g + j) * 3 * C + 16 * ct + i] = acc[ct][j];
    float *outo = PartO + (size_t)blockIdx.x * C * C;
#pragma unroll
    for (int ct = 0; ct < OT; ++ct)
#pragma unroll
        for (int j = 0; j < 4; ++j) outo[(size_t)(16 * w + 4 * g + j) * C + 16 * ct + i] = acco[ct][j];
}

// Tiles of k_bwd_proj per workgroup: all workgroups resident at once, two per compute unit.  Two groups of wavefronts share a
// workgroup (`halves`) from more than 256 tiles on.  Whole gradient with two groups and with one
// (us, k = 1): 294 tiles 53.9 / 58.4, 392 59.1 / 63.6, 490 65.5 / 70.8, 3136 207.0 / 216.5; below the line 49 tiles 32.5 / 31.8, 98 39.2 /
// 39.4, 196 47.2 / 47.3, 256 (16 x 32 x 32 x 64) 39.6 / 41.9: a line between 200 and 256 tiles would gain up to 5 % there.
struct ProjPlan {
    int tiles, per_wg, groups, halves;
};

ProjPlan proj_plan(long M)
{
    ProjPlan p;
    p.tiles = (int)((M + 63) / 64);
    p.per_wg = (p.tiles + 511) / 512;
    p.halves = p.tiles > 256 ? 2 : 1;
    p.per_wg *= p.halves;
    p.groups = (p.tiles + p.per_wg - 1) / p.per_wg;
    return p;
}

// One pass over the gradient map at C = 64; wider layers take the plain product for dX and shares of the tokens for both weight
// gradients: a workgroup that keeps all of dWqkv writes it once per compute unit, 50 MB of partial matrices at C = 128
// and their second reading.  Whole gradient in one pass and so (us): 64 x 56 x 56 x 64, k = 1 207 / 221, 32 images 118.9 / 121.2,
// 8 58.9 / 59.8, 4 47.2 / 46.6; 64 x 28 x 28 x 128, k = 4 160 / 139, 16 images 78.3 / 55.6, 4 47.1 / 35.7, 2 x 128 x 128 x 128,
// S = 16 158 / 131, one image of 14 x 14 x 128 34.7 / 26.2.
bool fused_projection(int C) { return C == 64; }

// Partial matrices of dWqkv and of dWo.
int weight_parts(long M, int C) { return fused_projection(C) ? proj_plan(M).groups : gemm_tn_shares(M, C, 3 * C, C, C); }

// Arrays of 25 C floats that the tap gradients come in.
int tap_parts(const Dims &D) { return attn_bwd_map_ok(D) && attn_bwd_map_convolves(D) ? D.B : lce::lce_grad_groups_bf16(D, 3 * D.C); }

struct BwdWs {
    bf16_t *q, *k, *v, *dO, *o, *dqkv;
    float *lse, *dsum, *part_qkv, *part_o, *part_lce;
    size_t bytes;
};

BwdWs carve_bwd(const Dims &D, void *ws)
{
    char *base = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += (bytes + 255) & ~(size_t)255;
        return p;
    };
    const long M = (long)D.B * D.N;
    const size_t MC = (size_t)M * D.C, C = D.C;
    BwdWs w;
    w.q = (bf16_t *)take(MC * 2);
    w.k = (bf16_t *)take(MC * 2);
    w.v = (bf16_t *)take(MC * 2);
    w.dO = (bf16_t *)take(MC * 2);
    w.o = (bf16_t *)take(MC * 2);
    w.dqkv = (bf16_t *)take(MC * 6);
    w.lse = (float *)take((size_t)M * D.heads * 4);
    w.dsum = (float *)take((size_t)M * D.heads * 4);
    const int parts = weight_parts(M, D.C);
    w.part_qkv = (float *)take((size_t)parts * 3 * C * C * 4);
    w.part_o = (float *)take((size_t)parts * C * C * 4);
    w.part_lce = (float *)take((size_t)tap_parts(D) * 25 * C * 4);
    w.bytes = off;
    return w;
}

bool launched() { return hipGetLastError() == hipSuccess; }

// Small maps of small regions go by whole images (Q as projected), everything else region by region (Q in units of log2).
// O = attention + LCE(V) (Eq. 7), dQ, dK, dV and the partial sums of the tap gradients.
int attention_and_lce(const Dims &D, const BwdWs &w, const int32_t *Ir, const bf16_t *Wlce, hipStream_t st)
{
    const lce::BackwardJobs L = lce::backward_jobs(D, w.dO, w.v, Wlce, w.o, w.dqkv + 2 * D.C, w.dqkv + D.C, 3 * D.C, w.part_lce);
    const AttnBwdArgs A = {w.q, w.k, w.v, w.dO, Ir, w.o, w.dqkv, w.lse, w.dsum};
    const bool map = attn_bwd_map_ok(D);
    const int rc = map ? launch_attn_bwd_map(D, w.q, w.k, w.v, w.dO, Ir, w.o, w.dqkv, Wlce, w.part_lce, K_GEN_BACKWARD, st) : launch_attn_bwd(D, A, L, K_GEN_BACKWARD, st);
    if (rc != BRA_OK || (map ? attn_bwd_map_convolves(D) : L.beside || attn_bwd_convolves(D, L))) return rc;
    return lce::lce_backward_bf16(D, L, K_GEN_BACKWARD, st);
}

// Images with more routing entries than this keep to the float32 kernels.
constexpr int kBwdMaxEntries = 4096;

}  // namespace

bool mfma_backward_supported(const Dims &D)
{
    static const bool off = experiment_flag("BRA_NO_MFMA_BACKWARD");
    if (off || D.dtype != BRA_BF16 || (D.d != 32 && D.d != 64) || D.C % 64 != 0 || D.C > 4096) return false;
    if ((long)D.R * D.k > kBwdMaxEntries || D.rh >= (1 << 20)) return false;
    const long M = (long)D.B * D.N;
    return M * 3 * D.C < (1L << 40) && (long)D.B * D.R * ((D.n + 63) / 64) * D.heads <= 0x7fffffffL &&
           M <= 0x7fffffffL;
}

size_t mfma_backward_workspace_bytes(const Dims &D) { return carve_bwd(D, nullptr).bytes; }

int mfma_backward(const Dims &D, const void *X, const void *Wqkv, const void *Wo, const void *Wlce,
                  const int32_t *Ir, const void *dY, void *dX, float *dWqkv, float *dWo, float *dWlce, void *ws,
                  hipStream_t st)
{
    const BwdWs w = carve_bwd(D, ws);
    const int C = D.C;
    const long M = (long)D.B * D.N;
    // Q, K, V once more (Eq. 3); dO = dY Wo^T
    const float q_scale = attn_bwd_map_ok(D) ? 1.0f : D.scale * 1.4426950408889634f;
    int rc = gemm_pair(GemmHalf{(const bf16_t *)X, (const bf16_t *)Wqkv, 3 * C, 3 * C, GemmOut{{w.q, w.k, w.v}, C, {nullptr, nullptr}, nullptr, nullptr, 0, q_scale}},
                       GemmHalf{(const bf16_t *)dY, (const bf16_t *)Wo, C, C, GemmOut{{w.dO, nullptr, nullptr}, C, {nullptr, nullptr}, nullptr, nullptr, 0}},
                       M, C, K_GEN_BACKWARD, st);
    if (rc != BRA_OK) return rc;
    rc = attention_and_lce(D, w, Ir, (const bf16_t *)Wlce, st);
    if (rc != BRA_OK) return rc;
    if (fused_projection(C)) {
        // dX = [dQ | dK | dV] Wqkv^T and the partial sums of dWqkv = X^T [dQ | dK | dV] and of dWo
        const ProjPlan pp = proj_plan(M);
        static bool opted[2] = {false, false};
        if (!(pp.halves == 2 ? opt_in(k_bwd_proj<2>, opted[1]) : opt_in(k_bwd_proj<1>, opted[0]))) return BRA_ERR_LAUNCH;
        ProfScope ps(st, K_GEN_BACKWARD);
        if (pp.halves == 2)
            hipLaunchKernelGGL(k_bwd_proj<2>, dim3(pp.groups), dim3(512), 2 * ProjSmem::bytes, st, w.dqkv, (const bf16_t *)X,
                               (const bf16_t *)Wqkv, (bf16_t *)dX, w.part_qkv, w.o, (const bf16_t *)dY, w.part_o, M, pp.tiles, pp.per_wg);
        else
            hipLaunchKernelGGL(k_bwd_proj<1>, dim3(pp.groups), dim3(256), ProjSmem::bytes, st, w.dqkv, (const bf16_t *)X,
                               (const bf16_t *)Wqkv, (bf16_t *)dX, w.part_qkv, w.o, (const bf16_t *)dY, w.part_o, M, pp.tiles, pp.per_wg);
        if (!launched()) return BRA_ERR_LAUNCH;
    } else {
        rc = gemm_bt_tn(GemmTn{(const bf16_t *)X, w.dqkv, w.part_qkv, C, 3 * C, C, 3 * C}, GemmTn{w.o, (const bf16_t *)dY, w.part_o, C, C, C, C},
                        GemmHalf{w.dqkv, (const bf16_t *)Wqkv, 3 * C, C, GemmOut{{dX, nullptr, nullptr}, C, {nullptr, nullptr}, nullptr, nullptr, 0}},
                        M, 3 * C, K_GEN_BACKWARD, st);
        if (rc != BRA_OK) return rc;
    }
    {
        const int parts = weight_parts(M, C);
        const ReduceJob j0 = reduce_job(w.part_qkv, dWqkv, parts, 3 * C * C);
        const ReduceJob j1 = reduce_job(w.part_o, dWo, parts, C * C);
        const ReduceJob j2 = reduce_job(w.part_lce, dWlce, tap_parts(D), 25 * C);
        ProfScope ps(st, K_GEN_BACKWARD);
        hipLaunchKernelGGL(k_reduce_parts, dim3(j0.blocks + j1.blocks + j2.blocks), dim3(256), 0, st, j0, j1, j2);
        if (!launched()) return BRA_ERR_LAUNCH;
    }
    return BRA_OK;
}

}  // namespace bra
