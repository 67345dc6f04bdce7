// Device-side kernels of the float32 family: products on v_mfma_f32_16x16x4_f32 (internal).
//
// Lane 16 g + i of that instruction holds A[row i][k g], B[k g][col i] and D[rows 4 g + j][col i].
// A lane that loads 4 consecutive values of the contraction axis feeds 4 such products: product e of
// step s then contracts over {16 s + 4 g' + e}, any order being right as long as both operands use the
// same one.  The float32 instruction runs at 64 flops per clock and SIMD, twice the vector unit without
// packed float32, and takes its operands 16 bytes per lane and 4 products, where a vector FMA reads LDS
// for every few flops: the vector kernels this replaces were bound by LDS reads and instruction issue.
//
// Every kernel takes float or bf16 tensors (template types) and any channel count; VEC selects 4-channel
// loads, for channel counts that are multiples of 4.
#pragma once

#include "bra_bwd_dev.h"
#include "bra_lce_dev.h"

#include <algorithm>
#include <type_traits>

namespace bra {
namespace f32 {

using mfma::bf16_hi;
using mfma::bf16_lo;
using mfma::cross_row_max;
using mfma::cross_row_sum;
using mfma::f32x2;
using mfma::f32x16;
using mfma::f32x4;
using mfma::kWave;
using mfma::divide;
using mfma::Places;
using mfma::u32x2;

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 4 consecutive elements as float32: p 16-byte (float) or 8-byte (bf16) aligned with VEC; without VEC
// elements past `left` read as zero.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float *p, int left)
{
    if (VEC) return *(const f32x4 *)p;
    return f32x4{left > 0 ? p[0] : 0.f, left > 1 ? p[1] : 0.f, left > 2 ? p[2] : 0.f, left > 3 ? p[3] : 0.f};
}
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const bf16_t *p, int left)
{
    if (VEC) {
        const u32x2 u = *(const u32x2 *)p;
        return f32x4{bf16_lo(u[0]), bf16_hi(u[0]), bf16_lo(u[1]), bf16_hi(u[1])};
    }
    return f32x4{left > 0 ? bf16_to_f32(p[0]) : 0.f, left > 1 ? bf16_to_f32(p[1]) : 0.f,
                 left > 2 ? bf16_to_f32(p[2]) : 0.f, left > 3 ? bf16_to_f32(p[3]) : 0.f};
}
template <bool VEC>
__device__ __forceinline__ void store4(float *p, f32x4 v, int left)
{
    if (VEC) { *(f32x4 *)p = v; return; }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < left) p[e] = v[e];
}
template <bool VEC>
__device__ __forceinline__ void store4(bf16_t *p, f32x4 v, int left)
{
    if (VEC) { *(u32x2 *)p = mfma::pack4(v); return; }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < left) p[e] = f32_to_bf16(v[e]);
}

// ---------------------------------------------------------------------------
// Out[m][n] = act(sum_k A[m][k] B[k][n] + bias[n]) + res[m][n] in float32, for a tile of 64 rows x BN
// columns per workgroup, the contraction in chunks of 32 staged in LDS (the next chunk is requested while
// the current one is multiplied).  The four wavefronts split the tile 2 x 2; the product is formed
// transposed (D[column 4 g + j][row i]), so that a lane stores 4 consecutive columns of one row.
// BT: B is read transposed (B[k][n] = Bm[n * ldb + k]).
// LDS pitches: 16-byte reads of 16 rows at 36 floats and 4-byte reads of 16 consecutive floats in 4 rows
// 4 pitches apart (BN + 4) both touch every bank once.
constexpr int kGemmBM = 64, kGemmBK = 32;

template <typename TA, typename TB, typename TO>
struct GemmJob {
    const TA *A;
    const TB *Bm;
    TO *Out;
    long M;
    int lda, ldb, ldo, N, K;
    const float *bias;
    const TO *res;          // the layout of Out
    int gelu;
};

// Rows taken region by region (n <= 64 tokens each) of maps of S x S regions of rh x rw tokens, a tile with 64 / n whole
// regions, and float32 means over each region's tokens of the first `cols` columns: [regions][cols].
struct MeansJob {
    float *Means;
    int cols, regions, R, S, n, rh, rw;
    float n_inv, R_inv, S_inv, rw_inv;
};

// The token of row `row` of tile `tile` (BM rows), or -1.
template <int BM = kGemmBM>
__device__ __forceinline__ int region_row(const MeansJob &g, int tile, int row)
{
    const int per = mfma::fast_div(BM, g.n_inv), first = tile * per, b0 = (unsigned)first / (unsigned)g.R, r0 = first - b0 * g.R;
    const int j = mfma::fast_div(row, g.n_inv), t = row - j * g.n;
    if (j >= per || first + j >= g.regions) return -1;
    const int over = mfma::fast_div(r0 + j, g.R_inv), reg = r0 + j - over * g.R;
    const int ry = mfma::fast_div(reg, g.S_inv), ty = mfma::fast_div(t, g.rw_inv);
    return ((b0 + over) * g.S * g.rh + ry * g.rh + ty) * g.S * g.rw + (reg - ry * g.S) * g.rw + t - ty * g.rw;
}

// The means of a tile's columns out of its accumulators: sums over aligned groups of 16 or 4 rows in registers (mfma::quad_sums: the
// quad's lanes end with the four columns of one 16 x 16 product each), where that is less than a region the groups, or with an odd
// number of rows all of them, meet in LDS.  The order does not depend on the tile's width.  sums: 64 x (BN + 4) floats.
template <int BN>
__device__ __forceinline__ void tile_means(const MeansJob &g, const f32x4 (&acc)[2][BN / 32], int tile, int n0, int N, float *sums)
{
    constexpr int MP = BN + 4, GROUPS = BN / 4, TR = 256 / GROUPS;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, lg = lane / 16, i = lane % 16, wr = wave / 2, wc = wave % 2;
    const int per = mfma::fast_div(kGemmBM, g.n_inv), first = tile * per, cols = min(g.cols, N);
    auto lay_down = [&](auto group) {
        constexpr int G = decltype(group)::value;
        const bool whole = G == g.n;
        if (!whole) __syncthreads();              // the last chunk has been read
#pragma unroll
        for (int t0 = 0; t0 < BN / 32; t0 += 2) {
            if constexpr (G == 1) {
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                    for (int t = t0; t < t0 + 2; ++t) {
                        const int row = 32 * wr + 16 * rt + i, col = (BN / 2) * wc + 16 * t + 4 * lg, region = tile * kGemmBM + row;
                        if (!whole) *(f32x4 *)(sums + row * MP + col) = acc[rt][t];
                        else if (n0 + col < cols && region < g.regions) *(f32x4 *)(g.Means + (size_t)region * g.cols + n0 + col) = acc[rt][t];
                    }
                continue;
            }
            f32x16 v;
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = acc[e / 8][t0 + e / 4 % 2][e % 4];
            f32x4 quad = mfma::quad_sums(v, i);
            if constexpr (G == 16)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    quad[e] += mfma::dpp_get<0x124>(quad[e]);       // row_ror:4
                    quad[e] += mfma::dpp_get<0x128>(quad[e]);       // row_ror:8
                }
            if (i % G >= 4) continue;
            const int row = 32 * wr + 16 * (i % 2) + i, col = (BN / 2) * wc + 16 * (t0 + i / 2 % 2) + 4 * lg, region = tile * (kGemmBM / G) + row / G;
            if (!whole) *(f32x4 *)(sums + row / G * MP + col) = quad;
            else if (n0 + col < cols && region < g.regions) *(f32x4 *)(g.Means + (size_t)region * g.cols + n0 + col) = quad * g.n_inv;
        }
    };
    const int G = mfma::means_group(g.n);
    if (G == 16) lay_down(std::integral_constant<int, 16>{});
    else if (G == 4) lay_down(std::integral_constant<int, 4>{});
    else lay_down(std::integral_constant<int, 1>{});
    if (G == g.n) return;
    __syncthreads();
    const int col = 4 * (tid % GROUPS), rows_each = g.n / G;
    for (int j = tid / GROUPS; j < per && first + j < g.regions; j += TR) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int t = 0; t < rows_each; ++t) sum += *(const f32x4 *)(sums + (j * rows_each + t) * MP + col);
        if (n0 + col < cols) *(f32x4 *)(g.Means + (size_t)(first + j) * g.cols + n0 + col) = sum * g.n_inv;
    }
}

// A wavefront's 32 rows from m0 on x BN / 2 columns from n0 on, with bias, GELU and residual.
// rows: if not NULL, the rows' tokens from the tile's row m0 on.
template <bool VEC, int BN, typename TA, typename TB, typename TO>
__device__ __forceinline__ void gemm_store(const GemmJob<TA, TB, TO> &J, const f32x4 (&acc)[2][BN / 32], long m0, int n0, int g, int i,
                                           const int *rows = nullptr)
{
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
        const long m = rows ? (long)rows[16 * rt + i] : m0 + 16 * rt + i;
        if (rows ? m < 0 : m >= J.M) continue;
#pragma unroll
        for (int t = 0; t < BN / 32; ++t) {
            const int n = n0 + 16 * t + 4 * g, left = J.N - n;
            if (left <= 0) continue;
            f32x4 v = acc[rt][t];
            if (J.bias) v += load4<VEC>(J.bias + n, left);
            if (J.gelu) v = f32x4{gelu_f32(v[0]), gelu_f32(v[1]), gelu_f32(v[2]), gelu_f32(v[3])};
            if (J.res) v += load4<VEC>(J.res + m * J.ldo + n, left);
            store4<VEC>(J.Out + m * J.ldo + n, v, left);
        }
    }
}

// MEANS: rows region by region, see MeansJob (M is not looked at); rows: a table of 64 in LDS.
template <bool BT, bool VEC, int BN, bool MEANS = false, typename TA, typename TB, typename TO>
__device__ __forceinline__ void gemm_tile(const GemmJob<TA, TB, TO> &J, int block, float *smem, const MeansJob *means = nullptr, int *rows = nullptr)
{
    constexpr int BK = kGemmBK, PA = BK + 4, PB = BT ? BK + 4 : BN + 4, NT = BN / 32;
    float *As = smem, *Bs = smem + kGemmBM * PA;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int ntiles = (J.N + BN - 1) / BN;
    const long m0 = (long)(block / ntiles) * kGemmBM;
    const int n0 = (block % ntiles) * BN;
    if (!MEANS && m0 >= J.M) return;             // grids are rounded up to multiples of 8
    if constexpr (MEANS) {
        if (tid < kGemmBM) rows[tid] = region_row(*means, block / ntiles, tid);
        __syncthreads();
    }
    constexpr int NA = kGemmBM * BK / 4 / 256, NB = BN * BK / 4 / 256;
    f32x4 ra[NA], rb[NB];
    // Rows past the end repeat the last one (never stored).  k past the end is blanked where the values go to LDS:
    // a select right behind the load would wait for it and take the prefetch away.
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int idx = tid + 256 * u, k = k0 + 4 * (idx % (BK / 4));
            const long m = MEANS ? (long)max(rows[idx / (BK / 4)], 0) : min(m0 + idx / (BK / 4), J.M - 1);
            ra[u] = load4<VEC>(J.A + m * J.lda + (VEC ? min(k, J.K - 4) : k), J.K - k);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int idx = tid + 256 * u;
            if (BT) {
                const int k = k0 + 4 * (idx % (BK / 4)), n = min(n0 + idx / (BK / 4), J.N - 1);
                rb[u] = load4<VEC>(J.Bm + (long)n * J.ldb + (VEC ? min(k, J.K - 4) : k), J.K - k);
            } else {
                const int k = k0 + idx / (BN / 4), n = n0 + 4 * (idx % (BN / 4));
                const TB *row = J.Bm + (long)min(k, J.K - 1) * J.ldb;
                rb[u] = load4<VEC>(row + (VEC ? min(n, J.N - 4) : n), J.N - n);
            }
        }
    };
    const int wr = wave / 2, wc = wave % 2;
    f32x4 acc[2][NT];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
    for (int k0 = 0; k0 < J.K; k0 += BK) {
        if (k0) __syncthreads();                 // the previous chunk has been read
        if (k0 + BK > J.K) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < NA; ++u)
                if (k0 + 4 * ((tid + 256 * u) % (BK / 4)) >= J.K) ra[u] = zero;
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (k0 + (BT ? 4 * ((tid + 256 * u) % (BK / 4)) : (tid + 256 * u) / (BN / 4)) >= J.K) rb[u] = zero;
        }
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int idx = tid + 256 * u;
            *(f32x4 *)(As + (idx / (BK / 4)) * PA + 4 * (idx % (BK / 4))) = ra[u];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int idx = tid + 256 * u;
            if (BT) *(f32x4 *)(Bs + (idx / (BK / 4)) * PB + 4 * (idx % (BK / 4))) = rb[u];
            else *(f32x4 *)(Bs + (idx / (BN / 4)) * PB + 4 * (idx % (BN / 4))) = rb[u];
        }
        __syncthreads();
        if (k0 + BK < J.K) fetch(k0 + BK);
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            f32x4 xb[2], wa[NT];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) xb[rt] = *(const f32x4 *)(As + (32 * wr + 16 * rt + i) * PA + 16 * s + 4 * g);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int n = (BN / 2) * wc + 16 * t + i;
                if (BT) wa[t] = *(const f32x4 *)(Bs + n * PB + 16 * s + 4 * g);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) wa[t][e] = Bs[(16 * s + 4 * g + e) * PB + n];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) acc[rt][t] = mfma_f32(wa[t][e], xb[rt][e], acc[rt][t]);
        }
    }
    if (!MEANS || J.Out) gemm_store<VEC, BN>(J, acc, m0 + 32 * wr, n0 + (BN / 2) * wc, g, i, MEANS ? rows + 32 * wr : nullptr);
    if (MEANS && n0 < means->cols) tile_means<BN>(*means, acc, block / ntiles, n0, J.N, smem);
}

// The same tile for a bf16 B, on v_mfma_f32_16x16x32_bf16, one step per chunk (the float32 instruction takes 16 times as
// long).  The products are those of the float32 numbers: a bf16 A enters as it is, a float32 A as three bf16 terms that
// add up to it exactly, smallest first.  Both operands lie in LDS as they came; B's rows (not BT) become an operand by the
// transposing read, 128 bytes more after every 8 of them keep its lane groups on different banks.  Channel counts are
// multiples of 4.  58310 x 96 x 288 with float32 results: 26 us (48 on the float32 instruction; 78 MB).
// 58310 x 96 x 96 with a float32 A 10.5 us (19.4).
template <bool BT, int BN, bool MEANS = false, typename TA, typename TO>
__device__ __forceinline__ void gemm_tile_bf16(const GemmJob<TA, bf16_t, TO> &J, int block, bf16_t *smem, const MeansJob *means = nullptr,
                                               int *rows = nullptr)
{
    using mfma::bf16x8;
    using mfma::u32x4;
    constexpr int BK = kGemmBK, PA = BK + 8, PB = BT ? BK + 8 : BN + 16, NT = BN / 32, NA = kGemmBM * BK / 4 / 256, NB = BN * BK / 4 / 256;
    constexpr bool SPLIT = std::is_same<TA, float>::value;
    constexpr int TERMS = SPLIT ? 3 : 1, plane = kGemmBM * PA;
    bf16_t *As = smem, *Bs = smem + TERMS * plane;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int ntiles = (J.N + BN - 1) / BN;
    const long m0 = (long)(block / ntiles) * kGemmBM;
    const int n0 = (block % ntiles) * BN;
    if (!MEANS && m0 >= J.M) return;             // grids are rounded up to multiples of 8
    if constexpr (MEANS) {
        if (block / ntiles * mfma::fast_div(kGemmBM, means->n_inv) >= means->regions) return;
        if (tid < kGemmBM) rows[tid] = region_row(*means, block / ntiles, tid);
        __syncthreads();
    }
    typename std::conditional<SPLIT, f32x4, u32x2>::type ra[NA];
    u32x2 rb[NB];
    auto fetch = [&](int k0) {               // past the end: as in gemm_tile
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int idx = tid + 256 * u, k = k0 + 4 * (idx % (BK / 4));
            const long m = MEANS ? (long)max(rows[idx / (BK / 4)], 0) : min(m0 + idx / (BK / 4), J.M - 1);
            ra[u] = *(const decltype(&ra[0]))(J.A + m * J.lda + min(k, J.K - 4));
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int idx = tid + 256 * u;
            if (BT) {
                const int k = k0 + 4 * (idx % (BK / 4)), n = min(n0 + idx / (BK / 4), J.N - 1);
                rb[u] = *(const u32x2 *)(J.Bm + (long)n * J.ldb + min(k, J.K - 4));
            } else {
                const int k = k0 + idx / (BN / 4), n = n0 + 4 * (idx % (BN / 4));
                rb[u] = *(const u32x2 *)(J.Bm + (long)min(k, J.K - 1) * J.ldb + min(n, J.N - 4));
            }
        }
    };
    const int wr = wave / 2, wc = wave % 2;
    f32x4 acc[2][NT];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
    for (int k0 = 0; k0 < J.K; k0 += BK) {
        if (k0) __syncthreads();                 // the previous chunk has been read
        if (k0 + BK > J.K) {
            const u32x2 zero = {0u, 0u};
#pragma unroll
            for (int u = 0; u < NA; ++u)
                if (k0 + 4 * ((tid + 256 * u) % (BK / 4)) >= J.K) ra[u] = {};
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (k0 + (BT ? 4 * ((tid + 256 * u) % (BK / 4)) : (tid + 256 * u) / (BN / 4)) >= J.K) rb[u] = zero;
        }
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int idx = tid + 256 * u;
            bf16_t *dst = As + (idx / (BK / 4)) * PA + 4 * (idx % (BK / 4));
            if constexpr (SPLIT) {
                f32x4 rest = ra[u];
#pragma unroll
                for (int q = 0; q < TERMS; ++q) {
                    const u32x2 term = mfma::pack4(rest);
                    *(u32x2 *)(dst + q * plane) = term;
                    rest -= f32x4{bf16_lo(term[0]), bf16_hi(term[0]), bf16_lo(term[1]), bf16_hi(term[1])};
                }
            } else {
                *(u32x2 *)dst = ra[u];
            }
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int idx = tid + 256 * u;
            if (BT) *(u32x2 *)(Bs + (idx / (BK / 4)) * PB + 4 * (idx % (BK / 4))) = rb[u];
            else *(u32x2 *)(Bs + (idx / (BN / 4)) * PB + idx / (BN / 4) / 8 * 64 + 4 * (idx % (BN / 4))) = rb[u];
        }
        __syncthreads();
        if (k0 + BK < J.K) fetch(k0 + BK);
        bf16x8 xb[2][TERMS];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int q = 0; q < TERMS; ++q) xb[rt][q] = *(const bf16x8 *)(As + q * plane + (32 * wr + 16 * rt + i) * PA + 8 * g);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int n = (BN / 2) * wc + 16 * t;
            bf16x8 wf;
            if (BT) {
                wf = *(const bf16x8 *)(Bs + (n + i) * PB + 8 * g);
            } else {
                const bf16_t *wp = Bs + (8 * g + i / 4) * PB + g * 64 + n + 4 * (i % 4);
                const u32x2 w0 = __builtin_bit_cast(u32x2, mfma::lds_read_tr16(wp)), w1 = __builtin_bit_cast(u32x2, mfma::lds_read_tr16(wp + 4 * PB));
                wf = __builtin_bit_cast(bf16x8, u32x4{w0[0], w0[1], w1[0], w1[1]});
            }
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int q = TERMS - 1; q >= 0; --q) acc[rt][t] = mfma::mfma16(wf, xb[rt][q], acc[rt][t]);
        }
    }
    if (!MEANS || J.Out) gemm_store<true, BN>(J, acc, m0 + 32 * wr, n0 + (BN / 2) * wc, g, i, MEANS ? rows + 32 * wr : nullptr);
    if (MEANS && n0 < means->cols) tile_means<BN>(*means, acc, block / ntiles, n0, J.N, (float *)smem);
}

template <int BN, bool BT>
constexpr size_t gemm_lds_floats()
{
    constexpr size_t f32 = (size_t)kGemmBM * (kGemmBK + 4) + (BT ? BN * (kGemmBK + 4) : kGemmBK * (BN + 4));
    constexpr size_t terms = (3 * (size_t)kGemmBM * (kGemmBK + 8) + (BT ? BN * (kGemmBK + 8) : kGemmBK * (BN + 16) + kGemmBK / 8 * 64)) / 2;
    return f32 > terms ? f32 : terms;
}

// Of `blocks` workgroups.  On the bf16 instruction, where memory is the bound, those of the same rows on one XCD (layer of 50 x 28 x 28 x 96
// bf16 76.0 -> 74.9 us, 62 x 16 x 16 x 96 56.5 -> 54.7); on the float32 one that was slower (2 x 64 x 64 x 128 49.4 -> 53.1).
template <bool BT, bool VEC, int BN, typename TA, typename TB, typename TO>
__device__ __forceinline__ void any_gemm_tile(const GemmJob<TA, TB, TO> &J, int block, int blocks, float *smem)
{
    if constexpr (VEC && std::is_same<TB, bf16_t>::value) gemm_tile_bf16<BT, BN>(J, mfma::swizzled(block, blocks), (bf16_t *)smem);
    else gemm_tile<BT, VEC, BN>(J, block, smem);
}

// Workgroups below blocks0 do job J0, the rest J1 (of the same B matrix type, A and Out float32): the
// region-level projection of the routing rides in the token projection's launch.
template <bool BT, bool VEC, int BN, typename TA, typename TB, typename TO>
__global__ __launch_bounds__(256) void k_gemm(GemmJob<TA, TB, TO> J0, GemmJob<float, TB, float> J1, int blocks0)
{
    __shared__ __attribute__((aligned(16))) float smem[gemm_lds_floats<BN, BT>()];
    if ((int)blockIdx.x < blocks0) any_gemm_tile<BT, VEC, BN>(J0, blockIdx.x, blocks0, smem);
    else any_gemm_tile<BT, VEC, BN>(J1, (int)blockIdx.x - blocks0, (int)gridDim.x - blocks0, smem);
}

// A product whose rows go region by region, with their means.
template <int BN, typename T>
__global__ __launch_bounds__(256) void k_gemm_means(GemmJob<T, T, float> J, MeansJob means)
{
    constexpr size_t n = gemm_lds_floats<BN, false>(), sums = (size_t)kGemmBM * (BN + 4);
    __shared__ __attribute__((aligned(16))) float smem[n > sums ? n : sums];
    __shared__ int rows[kGemmBM];
    if constexpr (std::is_same<T, bf16_t>::value) gemm_tile_bf16<false, BN, true>(J, mfma::swizzled_block(), (bf16_t *)smem, &means, rows);
    else gemm_tile<false, true, BN, true>(J, blockIdx.x, smem, &means, rows);
}

// J0 and a product with its matrix transposed (Q, K, V = X Wqkv and dO = dY Wo^T of the gradients) in one launch.
template <bool VEC, int BN, typename T>
__global__ __launch_bounds__(256) void k_gemm_both(GemmJob<T, T, float> J0, GemmJob<T, T, float> J1, int blocks0)
{
    constexpr size_t n0 = gemm_lds_floats<BN, false>(), n1 = gemm_lds_floats<BN, true>();
    __shared__ __attribute__((aligned(16))) float smem[n0 > n1 ? n0 : n1];
    if ((int)blockIdx.x < blocks0) any_gemm_tile<false, VEC, BN>(J0, blockIdx.x, blocks0, smem);
    else any_gemm_tile<true, VEC, BN>(J1, (int)blockIdx.x - blocks0, (int)gridDim.x - blocks0, smem);
}

// Few rows: a tile of 16 RT rows x 32 columns per workgroup, whose wavefronts share the contraction and add up through LDS in a fixed
// order.  The tiles above leave most of the chip idle there and walk the whole contraction with one wavefront per SIMD, 0.75 us for
// 32 of it; here operands come straight from memory, four steps of 16 ahead, and nothing is waited for in between.
// Whole tiles of columns and of steps (N % 32 = K % 16 = 0).  BT, MEANS: as above (n <= 16 RT).
constexpr int kSplitPitch = 36;          // floats per row of partial sums
template <int RT, int WAVES>
constexpr size_t split_lds_floats() { return (size_t)WAVES * 16 * RT * kSplitPitch; }

template <bool BT, int RT, int WAVES, bool MEANS = false>
__device__ __forceinline__ void split_tile(const GemmJob<float, float, float> &J, int block, float *smem, const MeansJob *means = nullptr, int *rows = nullptr)
{
    constexpr int BM = 16 * RT, AHEAD = 4, P = kSplitPitch;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int ntiles = J.N / 32, tile = block / ntiles, n0 = 32 * (block - tile * ntiles);
    const long m0 = (long)tile * BM;
    if constexpr (MEANS) {
        if (tid < BM) rows[tid] = region_row<BM>(*means, tile, tid);
        __syncthreads();
    }
    const int steps = J.K / 16, s0 = steps * wave / WAVES, s1 = steps * (wave + 1) / WAVES;
    const float *a[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) a[rt] = J.A + (MEANS ? (long)max(rows[16 * rt + i], 0) : min(m0 + 16 * rt + i, J.M - 1)) * J.lda + 4 * g;
    const float *b = BT ? J.Bm + (long)(n0 + i) * J.ldb + 4 * g : J.Bm + (long)(4 * g) * J.ldb + n0 + 2 * i;
    const long bstep = BT ? 16 : 16L * J.ldb;
    f32x4 ra[2][AHEAD][RT], rb[2][AHEAD][2];     // [t]: k 4 g .. 4 g + 3 of column 16 t + i (BT) or 2 i + t
    auto fetch = [&](int s, f32x4 (&x)[AHEAD][RT], f32x4 (&w)[AHEAD][2]) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int at = min(s + u, steps - 1);        // past the end: not used
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) x[u][rt] = *(const f32x4 *)(a[rt] + 16 * at);
            const float *p = b + at * bstep;
            if (BT) {
                w[u][0] = *(const f32x4 *)p;
                w[u][1] = *(const f32x4 *)(p + 16L * J.ldb);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x2 v = *(const f32x2 *)(p + (long)e * J.ldb);
                    w[u][0][e] = v[0];
                    w[u][1][e] = v[1];
                }
            }
        }
    };
    f32x4 acc[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt][0] = acc[rt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto work = [&](int s, const f32x4 (&x)[AHEAD][RT], const f32x4 (&w)[AHEAD][2]) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (s + u >= s1) break;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) acc[rt][t] = mfma_f32(w[u][t][e], x[u][rt][e], acc[rt][t]);
        }
    };
    if (s0 < s1) fetch(s0, ra[0], rb[0]);
    for (int s = s0; s < s1; s += 2 * AHEAD) {
        if (s + AHEAD < s1) fetch(s + AHEAD, ra[1], rb[1]);
        work(s, ra[0], rb[0]);
        if (s + AHEAD >= s1) break;
        if (s + 2 * AHEAD < s1) fetch(s + 2 * AHEAD, ra[0], rb[0]);
        work(s + AHEAD, ra[1], rb[1]);
    }
    float *mine = smem + wave * BM * P;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        float *to = mine + (16 * rt + i) * P;
        const f32x4 v0 = acc[rt][0], v1 = acc[rt][1];
        *(f32x4 *)(to + (BT ? 4 * g : 8 * g)) = BT ? v0 : f32x4{v0[0], v1[0], v0[1], v1[1]};
        *(f32x4 *)(to + (BT ? 16 + 4 * g : 8 * g + 4)) = BT ? v1 : f32x4{v0[2], v1[2], v0[3], v1[3]};
    }
    __syncthreads();
    for (int e = tid; e < 8 * BM; e += 64 * WAVES) {
        const int row = e / 8, n = n0 + 4 * (e % 8);
        float *at = smem + row * P + 4 * (e % 8);
        f32x4 v = *(const f32x4 *)at;
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v += *(const f32x4 *)(at + w * BM * P);
        if (MEANS) *(f32x4 *)at = v;
        const long m = MEANS ? (long)rows[row] : m0 + row;
        if ((MEANS ? m < 0 : m >= J.M) || (MEANS && !J.Out)) continue;
        if (J.bias) v += *(const f32x4 *)(J.bias + n);
        if (J.gelu) v = f32x4{gelu_f32(v[0]), gelu_f32(v[1]), gelu_f32(v[2]), gelu_f32(v[3])};
        if (J.res) v += *(const f32x4 *)(J.res + m * J.ldo + n);
        *(f32x4 *)(J.Out + m * J.ldo + n) = v;
    }
    if constexpr (MEANS) {
        if (n0 >= means->cols) return;
        __syncthreads();
        const int n = means->n, per = mfma::fast_div(BM, means->n_inv), first = tile * per;
        for (int e = tid; e < 8 * per; e += 64 * WAVES) {
            const int j = e / 8;
            if (first + j >= means->regions) break;
            const float *at = smem + j * n * P + 4 * (e % 8);
            f32x4 sum = *(const f32x4 *)at;
            for (int t = 1; t < n; ++t) sum += *(const f32x4 *)(at + t * P);
            *(f32x4 *)(means->Means + (size_t)(first + j) * means->cols + n0 + 4 * (e % 8)) = sum * means->n_inv;
        }
    }
}

template <bool BT, int RT>
__global__ __launch_bounds__(512) void k_gemm_split(GemmJob<float, float, float> J)
{
    __shared__ __attribute__((aligned(16))) float smem[split_lds_floats<RT, 8>()];
    split_tile<BT, RT, 8>(J, blockIdx.x, smem);
}

template <int RT>
__global__ __launch_bounds__(512) void k_gemm_means_split(GemmJob<float, float, float> J, MeansJob means)
{
    __shared__ __attribute__((aligned(16))) float smem[split_lds_floats<RT, 8>()];
    __shared__ int rows[16 * RT];
    split_tile<false, RT, 8, true>(J, blockIdx.x, smem, &means, rows);
}

template <int RT>
__global__ __launch_bounds__(512) void k_gemm_both_split(GemmJob<float, float, float> J0, GemmJob<float, float, float> J1, int blocks0)
{
    __shared__ __attribute__((aligned(16))) float smem[split_lds_floats<RT, 8>()];
    if ((int)blockIdx.x < blocks0) split_tile<false, RT, 8>(J0, blockIdx.x, smem);
    else split_tile<true, RT, 8>(J1, (int)blockIdx.x - blocks0, smem);
}

// ---------------------------------------------------------------------------
// Xr[b, r, :] = mean over the n tokens of region r.  SUB (a power of two up to 64) consecutive lanes share
// one (image, region, 4-channel chunk): lane s adds tokens s, s + SUB, .. of the region (row-major), then
// the partial sums are combined pairwise in a fixed order.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_pool(const T *__restrict__ X, float *__restrict__ Xr, Dims D, int SUB)
{
    const int CH = (D.C + 3) / 4;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const long total = (long)D.B * D.R * CH, item = min(idx / SUB, total - 1);
    const int sub = (int)(idx % SUB);
    const int cc = (int)(item % CH), r = (int)((item / CH) % D.R), b = (int)(item / ((long)CH * D.R));
    const T *base = X + (((size_t)b * D.H + (r / D.S) * D.rh) * D.W + (r % D.S) * D.rw) * D.C + 4 * cc;
    const float rw_inv = 1.0f / (float)D.rw;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int slot = sub; slot < D.n; slot += SUB) {
        const int y = D.rh < (1 << 20) ? divide(slot, D.rw, rw_inv) : slot / D.rw, x = slot - y * D.rw;
        acc += load4<VEC>(base + ((size_t)y * D.W + x) * D.C, D.C - 4 * cc);
    }
    for (int off = 1; off < SUB; off *= 2)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off);
    if (idx / SUB < total && sub == 0) store4<VEC>(Xr + ((size_t)b * D.R + r) * D.C + 4 * cc, acc * (1.0f / (float)D.n), D.C - 4 * cc);
}

// ---------------------------------------------------------------------------
// Routed attention (Eq. 6, Eq. 1) in float32 for heads of at most DP (32 or 64) channels; QKV is
// [B, N, 3C] (q | k | v per token).  Workgroup (image, region, query tile, HPW heads): wavefront w has the
// head w / (4 / HPW) of the group and 16 queries; regions of at most 16 tokens put four heads side by
// side, larger ones 64 queries of one head.  The k n routed keys are taken KB at a time: their K and V rows
// (found by index in the projected map; no gathered tensor) go to LDS, the next block being requested
// meanwhile; S^T = K Q^T (a lane ends with 4 consecutive keys of one query), one online softmax over all
// routed keys, O^T += V^T P^T with the weights straight from the registers they were formed in.
// Head channels past d are zero on both sides.
template <int DP, int HPW>
struct AttnShape {
    static constexpr int CW = DP * HPW, P = CW + 4, KB = CW <= 64 ? 64 : 32, TPH = 4 / HPW, QT = 16 * TPH;
};

// Rows of a token map -> registers: channels of the workgroup's HPW heads, 4 at a time; head h0 + hl owns
// channels [(h0 + hl) d, (h0 + hl + 1) d).
// With VEC a chunk past the end reads the row's first channels: blank it with head_chunk_ok where it is used, not
// right behind the load (that would wait for it).
template <int DP>
__device__ __forceinline__ int head_chunk_left(int c4, int h0, const Dims &D)
{
    return h0 + 4 * c4 / DP < D.heads ? D.d - (4 * c4) % DP : 0;
}
template <int DP, bool VEC>
__device__ __forceinline__ f32x4 load_head_chunk(const float *row, int c4, int h0, const Dims &D)
{
    const int left = head_chunk_left<DP>(c4, h0, D);
    return load4<VEC>(row + (left > 0 ? (h0 + 4 * c4 / DP) * D.d + (4 * c4) % DP : 0), left);
}
template <int DP, bool VEC>
__device__ __forceinline__ f32x4 blank_head_chunk(f32x4 v, int c4, int h0, const Dims &D)
{
    return !VEC || head_chunk_left<DP>(c4, h0, D) > 0 ? v : f32x4{0.f, 0.f, 0.f, 0.f};
}

// acc[dt] += T^T x w: T's rows 16 t + 4 g + e (T points at row 4 g, column i) against the weights w[t][e], columns 16 dt + i.
// The operands of the next 16 rows are on their way while this tile's products run.
template <int KT, int NS>
__device__ __forceinline__ void rows_product(const float *T, int P, const f32x4 (&w)[KT], f32x4 (&acc)[NS])
{
    float v[2][4][NS];
    auto load = [&](int t) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) v[t % 2][e][dt] = T[(16 * t + e) * P + 16 * dt];
    };
    load(0);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        if (t + 1 < KT) load(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) acc[dt] = mfma_f32(v[t % 2][e][dt], w[t][e], acc[dt]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// One block of KB keys: scores, softmax, weights times V.  Kw, Vw: this wavefront's head in the rows of K and V (pitch P); m: reference score; l:
// this lane's part of the denominator; left: keys there are.
template <int KB, int P, int NS>
__device__ __forceinline__ void attention_block(const float *Kw, const float *Vw, const f32x4 (&qf)[NS], int left, bool begins, int g, int i, float &m,
                                                float (&l)[4], f32x4 (&acc)[NS])
{
    constexpr int KT = KB / 16;
    f32x4 st[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) st[t] = f32x4{-m, -m, -m, -m};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        f32x4 kf[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) kf[t] = *(const f32x4 *)(Kw + (16 * t + i) * P + 16 * s + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < KT; ++t) st[t] = mfma_f32(kf[t][e], qf[s][e], st[t]);   // S^T[key 16 t + 4 g + j][query i] - m
    }
    if (left < KB) {
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[t][j] = 16 * t + 4 * g + j < left ? st[t][j] : -INFINITY;
    }
    float mx = st[0][0];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) mx = fmaxf(mx, st[t][j]);
    // the reference follows the maximum when a lane's own score exceeds it by 2^8; the quotient does not depend on it
    if (begins || __builtin_amdgcn_ballot_w64(mx > 8.0f) != 0) {
        const float up = begins ? cross_row_max(mx) : fmaxf(cross_row_max(mx), 0.f);
        m += up;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[t][j] -= up;
        if (!begins) {
            const float alpha = __builtin_amdgcn_exp2f(-up);
#pragma unroll
            for (int j = 0; j < 4; ++j) l[j] *= alpha;
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) acc[dt] *= alpha;
        }
    }
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            st[t][j] = __builtin_amdgcn_exp2f(st[t][j]);
            l[j] += st[t][j];
        }
    rows_product<KT, NS>(Vw + 4 * g * P + i, P, st, acc);
}

// What a workgroup of the attention works on.  by_image: those of an image and head group on one XCD, whose L2 then holds that
// pair's rows (attention_by_image(), gradients_by_image()); else the head groups of a region next to each other, on different ones.
struct AttnWork {
    int tile, region, hg, image;
};

__device__ __forceinline__ AttnWork attn_work(int block, int blocks, bool by_image, int tiles, int hgroups, int R)
{
    const int at = by_image ? mfma::swizzled(block, blocks) : block, n0 = by_image ? tiles : hgroups, n1 = by_image ? R : tiles, n2 = by_image ? hgroups : R;
    const int q0 = at / n0, r0 = at - q0 * n0, q1 = q0 / n1, r1 = q0 - q1 * n1, image = q1 / n2, r2 = q1 - image * n2;
    return by_image ? AttnWork{r0, r1, r2, image} : AttnWork{r1, r2, r0, image};
}

// HPW = 1: as many wavefronts as the region's query tiles of 16 fill (3 to 8; more tiles are dealt out evenly).
// OUT: with Y = O Wo (Eq. 7) for the four heads of C = 128 and regions of at most 16 tokens; O, which holds LCE(V), is read and not written.  A
// wavefront forms 32 columns of Y, lane i's operands of two tiles being neighbours in a row of Wo.
template <int DP, int HPW, bool VEC, bool OUT = false>
__global__ __launch_bounds__(HPW == 1 ? 512 : 256, DP == 32 ? 4 : 2) void k_attention(const float *__restrict__ QKV, const int32_t *__restrict__ Ir,
                                                   float *__restrict__ O, Dims D, int hgroups, int qtiles, bool by_image, bool adds, const float *__restrict__ Wo, float *__restrict__ Y)
{
    static_assert(!OUT || (DP == 32 && HPW == 4 && VEC), "C = 128");
    typedef AttnShape<DP, HPW> L;
    constexpr int P = L::P, KB = L::KB, CW = L::CW, NS = DP / 16;
    __shared__ __attribute__((aligned(16))) float Ks[KB * P];
    __shared__ __attribute__((aligned(16))) float Vs[KB * P];
    const AttnWork work = attn_work(blockIdx.x, gridDim.x, by_image, qtiles, hgroups, D.R);
    const int qt = work.tile, reg = work.region, hg = work.hg, b = work.image;
    if (b >= D.B) return;
    const int T = HPW == 1 ? (int)blockDim.x : 256, tph = HPW == 1 ? T / kWave : L::TPH;      // query tiles
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int C3 = 3 * D.C, kn = D.kn, hl = HPW == 1 ? 0 : wave / L::TPH, h = hg * HPW + hl;
    const float *img = QKV + (size_t)b * D.N * C3;
    const int32_t *irp = Ir + ((size_t)b * D.R + reg) * D.k;
    const int slot0 = 16 * (tph * qt + (HPW == 1 ? wave : wave % L::TPH)), slot = slot0 + i;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n;
    const int qtok = at.origin(reg) + at.slot(min(slot, D.n - 1));
    f32x4 qf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        qf[s] = blank_head_chunk<DP, VEC>(load_head_chunk<DP, VEC>(img + (size_t)qtok * C3, 4 * s + g, h, D), 4 * s + g, h, D);

    constexpr int CHUNKS = KB * CW / 4, NL = HPW == 1 ? (CHUNKS + 191) / 192 : CHUNKS / 256;
    f32x4 kr[NL], vr[NL];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            if (HPW == 1 && u && T * u >= CHUNKS) break;
            const int idx = HPW == 1 ? min(tid + T * u, CHUNKS - 1) : tid + T * u;
            const int key = min(k0 + idx / (CW / 4), kn - 1);   // past the end: the last key, masked below
            const int p = divide(key, D.n, n_inv);
            const float *row = img + (size_t)(at.origin(region_index(irp[p], D.R)) + at.slot(key - p * D.n)) * C3;
            kr[u] = load_head_chunk<DP, VEC>(row + D.C, idx % (CW / 4), hg * HPW, D);
            vr[u] = load_head_chunk<DP, VEC>(row + 2 * D.C, idx % (CW / 4), hg * HPW, D);
        }
    };
    float m = 0.f, l[4] = {0.f, 0.f, 0.f, 0.f};      // reference score; this lane's part of the denominator
    f32x4 acc[NS];
#pragma unroll
    for (int dt = 0; dt < NS; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float c_exp = D.scale * 1.4426950408889634f;
#pragma unroll
    for (int s = 0; s < NS; ++s) qf[s] *= c_exp;     // scores as exponents of 2
    const bool idle = slot0 >= D.n || h >= D.heads;
    fetch(0);
    for (int k0 = 0; k0 < kn; k0 += KB) {
        if (k0) __syncthreads();                 // the previous block has been read
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tid + T * u;
            if (HPW == 1 && idx >= CHUNKS) break;
            *(f32x4 *)(Ks + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(kr[u], idx % (CW / 4), hg * HPW, D);
            *(f32x4 *)(Vs + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(vr[u], idx % (CW / 4), hg * HPW, D);
        }
        __syncthreads();
        if (k0 + KB < kn) fetch(k0 + KB);
        if (idle) continue;                      // no queries: the wavefront only brings its rows
        attention_block<KB, P, NS>(Ks + DP * hl, Vs + DP * hl, qf, kn - k0, k0 == 0, g, i, m, l, acc);
    }
    const float denominator = cross_row_sum((l[0] + l[1]) + (l[2] + l[3]));
    if constexpr (OUT) {
        const float inv = 1.0f / denominator, *added = O + ((size_t)b * D.N + qtok) * CW + DP * hl + 4 * g;
        __syncthreads();                         // the last block has been read
#pragma unroll
        for (int dt = 0; dt < NS; ++dt) {
            f32x4 v = acc[dt] * inv;
            v += *(const f32x4 *)(added + 16 * dt);
            *(f32x4 *)(Ks + i * P + DP * hl + 16 * dt + 4 * g) = v;
        }
        __syncthreads();
        const float *w = Wo + (size_t)4 * g * CW + 32 * wave + 2 * i;
        f32x4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < CW / 16; ++s) {
            const f32x4 x = *(const f32x4 *)(Ks + i * P + 16 * s + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x2 v = *(const f32x2 *)(w + (size_t)(16 * s + e) * CW);
#pragma unroll
                for (int t = 0; t < 2; ++t) y[t] = mfma_f32(v[t], x[e], y[t]);
            }
        }
        if (slot >= D.n) return;
        float *to = Y + ((size_t)b * D.N + qtok) * CW + 32 * wave + 8 * g;      // columns 8 g + 2 j + t
        *(f32x4 *)to = f32x4{y[0][0], y[1][0], y[0][1], y[1][1]};
        *(f32x4 *)(to + 4) = f32x4{y[0][2], y[1][2], y[0][3], y[1][3]};
        return;
    }
    if (slot < D.n && h < D.heads) {
        const float inv = 1.0f / denominator;
        float *orow = O + ((size_t)b * D.N + qtok) * D.C + h * D.d;
#pragma unroll
        for (int dt = 0; dt < NS; ++dt) {
            const int ch = 16 * dt + 4 * g;
            if (ch >= D.d) continue;
            f32x4 v = acc[dt] * inv;
            if (adds) v += load4<VEC>(orow + ch, D.d - ch);      // LCE(V)
            store4<VEC>(orow + ch, v, D.d - ch);
        }
    }
}

// The same for both heads of 32 channels of C = 64, with Y = O Wo (Eq. 7) behind it: O, which holds LCE(V), is read and not written.  Of
// 2 tph wavefronts w has head w / tph and queries 16 (w % tph) on, then 16 rows and 32 columns of Y.  The additions of Y are gemm_tile's.
// NL: chunks of a thread; 4 for 4 wavefronts, 2 for 8 and more.
// 16 x 56 x 56, k = 1: 24 us, 19 and 9.5 for the two apart, of 126 registers and four wavefronts per SIMD: bound by what hides the chain of a
// block of keys, loads, scores, weights, products and a barrier, with a round and a half of workgroups.
constexpr size_t out_lds_bytes(int tph) { return (size_t)std::max(2 * 64, 16 * tph + 64) * (64 + 4) * sizeof(float); }

template <int NL>
__global__ __launch_bounds__(NL == 4 ? 256 : 1024, 4) void k_attention_out(const float *__restrict__ QKV, const int32_t *__restrict__ Ir, const float *__restrict__ O,
                                                          const float *__restrict__ Wo, float *__restrict__ Y, Dims D, int qtiles)
{
    constexpr int C = 64, C3 = 3 * C, P = C + 4, KB = 64, NS = 2;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *Ks = smem, *Vs = smem + KB * P;
    const int block = mfma::swizzled_block(), qt = block % qtiles, reg = (block / qtiles) % D.R, b = block / (qtiles * D.R);
    if (b >= D.B) return;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int T = blockDim.x, tph = T / (2 * kWave), hl = wave >= tph, mine = wave - hl * tph, slot0 = 16 * (tph * qt + mine), kn = D.kn;
    const float *img = QKV + (size_t)b * D.N * C3;
    const int32_t *irp = Ir + ((size_t)b * D.R + reg) * D.k;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n;
    auto token = [&](int slot) { return at.origin(reg) + at.slot(min(slot, D.n - 1)); };
    const float c_exp = D.scale * 1.4426950408889634f;
    f32x4 qf[NS];
    {
        const float *row = img + (size_t)token(slot0 + i) * C3 + 32 * hl + 4 * g;
#pragma unroll
        for (int s = 0; s < NS; ++s) qf[s] = *(const f32x4 *)(row + 16 * s) * c_exp;      // scores as exponents of 2
    }
    // a thread's chunks of 4 channels: chunk tid % 16 of every (T / 16)th of 64 rows from tid / 16 on
    f32x4 kr[NL], vr[NL];
    const int ch = 4 * (tid % 16), r0 = tid / 16, rows = T / 16;
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int key = min(k0 + min(r0 + rows * u, KB - 1), kn - 1), p = divide(key, D.n, n_inv);   // past the end: the last key, masked below
            const float *row = img + (size_t)(at.origin(region_index(irp[p], D.R)) + at.slot(key - p * D.n)) * C3 + ch;
            kr[u] = *(const f32x4 *)(row + C);
            vr[u] = *(const f32x4 *)(row + 2 * C);
        }
    };
    auto park = [&](float *to, const f32x4 (&r)[NL]) {
#pragma unroll
        for (int u = 0; u < NL; ++u)
            if (r0 + rows * u < KB) *(f32x4 *)(to + (r0 + rows * u) * P + ch) = r[u];
    };
    float m = 0.f, l[4] = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[NS] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    fetch(0);
    for (int k0 = 0; k0 < kn; k0 += KB) {
        if (k0) __syncthreads();                 // the previous block has been read
        park(Ks, kr);
        park(Vs, vr);
        __syncthreads();
        if (k0 + KB < kn) fetch(k0 + KB);
        else {                                   // what the end needs: LCE(V) of the queries, two rows per thread, and Wo
#pragma unroll
            for (int u = 0; u < 2; ++u) kr[u] = *(const f32x4 *)(O + ((size_t)b * D.N + token(16 * tph * qt + r0 + rows * u)) * C + ch);
#pragma unroll
            for (int u = 0; u < NL; ++u) vr[u] = *(const f32x4 *)(Wo + min(r0 + rows * u, KB - 1) * C + ch);
        }
        if (slot0 < D.n) attention_block<KB, P, NS>(Ks + 32 * hl, Vs + 32 * hl, qf, kn - k0, k0 == 0, g, i, m, l, acc);
    }
    const float inv = 1.0f / cross_row_sum((l[0] + l[1]) + (l[2] + l[3]));
    float *Os = smem, *Ws = smem + 16 * tph * P;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) *(f32x4 *)(Os + (r0 + rows * u) * P + ch) = kr[u];
    park(Ws, vr);
    __syncthreads();
#pragma unroll
    for (int dt = 0; dt < NS; ++dt) {
        float *o = Os + (16 * mine + i) * P + 32 * hl + 16 * dt + 4 * g;
        f32x4 v = acc[dt] * inv;
        v += *(const f32x4 *)o;
        *(f32x4 *)o = v;
    }
    __syncthreads();
    const int rt = wave / 2, n0 = 32 * (wave % 2), slot = 16 * (tph * qt + rt) + i;
    f32x4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < C / 16; ++s) {
        const f32x4 x = *(const f32x4 *)(Os + (16 * rt + i) * P + 16 * s + 4 * g);
        float w[4][2];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 2; ++t) w[e][t] = Ws[(16 * s + 4 * g + e) * P + n0 + 16 * t + i];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 2; ++t) y[t] = mfma_f32(w[e][t], x[e], y[t]);
    }
    if (slot >= D.n) return;
    float *to = Y + ((size_t)b * D.N + token(slot)) * C + n0 + 4 * g;
#pragma unroll
    for (int t = 0; t < 2; ++t) *(f32x4 *)(to + 16 * t) = y[t];
}

// ---------------------------------------------------------------------------
// Query side of the attention backward (derivative of Eq. 6 with Eq. 1) in float32: the workgroup's queries
// and head groups as in k_attention.  First sweep over the key blocks, with the online softmax's rescaling:
// the maximum m, l = sum e, O~ = sum e V and D~ = sum e dP (dP^T = V dO^T); at its end O, D = D~ / l and
// lse = log2(l) + scale log2(e) m are final.  Second sweep: P = exp2(scale log2(e) s - lse),
// dS = P (dP - D), dQ^T += K^T dS^T.  A single key block (k n <= KB) is not taken twice.
template <int DP, int HPW, bool VEC>
__global__ __launch_bounds__(256) void k_attn_bwd_q(const float *__restrict__ QKV, const float *__restrict__ dO,
                                                    const int32_t *__restrict__ Ir, float *__restrict__ O,
                                                    float *__restrict__ dQKV, float *__restrict__ lse,
                                                    float *__restrict__ dsum, Dims D, int hgroups, int qtiles, bool by_image,
                                                    lce::GradJob<float> J, int lce_blocks)
{
    typedef AttnShape<DP, HPW> L;
    constexpr int P = L::P, CW = L::CW, KB = L::KB, KT = KB / 16, NS = DP / 16, kFloats = 2 * KB * P > 25 * 256 ? 2 * KB * P : 25 * 256;
    __shared__ __attribute__((aligned(16))) float lds[kFloats];
    float *Ks = lds, *Vs = lds + KB * P;
    int wg, wgs;
    if (lce::block_of_pass(lce_blocks, false, wg, wgs)) {
        lce::lce_grad_block<VEC ? 2 : 1, false>(J, D, mfma::swizzled(wg, wgs), lds);
        return;
    }
    const AttnWork work = attn_work(wg, wgs, by_image, qtiles, hgroups, D.R);
    const int qt = work.tile, reg = work.region, hg = work.hg, b = work.image;
    if (b >= D.B) return;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int C3 = 3 * D.C, kn = D.kn, nblocks = (kn + KB - 1) / KB, hl = wave / L::TPH, h = hg * HPW + hl;
    const size_t itok = (size_t)b * D.N;
    const float *img = QKV + itok * C3;
    const int32_t *irp = Ir + ((size_t)b * D.R + reg) * D.k;
    const int slot = L::QT * qt + 16 * (wave % L::TPH) + i;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n;
    const int qtok = at.origin(reg) + at.slot(min(slot, D.n - 1));
    const bool live = slot < D.n && h < D.heads;
    f32x4 qf[NS], gf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        qf[s] = blank_head_chunk<DP, VEC>(load_head_chunk<DP, VEC>(img + (size_t)qtok * C3, 4 * s + g, h, D), 4 * s + g, h, D);
        gf[s] = blank_head_chunk<DP, VEC>(load_head_chunk<DP, VEC>(dO + (itok + qtok) * D.C, 4 * s + g, h, D), 4 * s + g, h, D);
    }
    constexpr int NL = KB * CW / 4 / 256;
    f32x4 kr[NL], vr[NL];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tid + 256 * u, key = min(k0 + idx / (CW / 4), kn - 1);   // past the end: the last key, masked below
            const int p = divide(key, D.n, n_inv);
            const float *row = img + (size_t)(at.origin(region_index(irp[p], D.R)) + at.slot(key - p * D.n)) * C3;
            kr[u] = load_head_chunk<DP, VEC>(row + D.C, idx % (CW / 4), hg * HPW, D);
            vr[u] = load_head_chunk<DP, VEC>(row + 2 * D.C, idx % (CW / 4), hg * HPW, D);
        }
    };
    float m = -INFINITY, l = 0.f, dd = 0.f;
    f32x4 acc[NS];
#pragma unroll
    for (int dt = 0; dt < NS; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float c_exp = D.scale * 1.4426950408889634f;
    // acc[dt] = T^T[channel 16 dt + 4 g + j][..] x weights of the block's keys
    auto contract = [&](const float *T, const f32x4 (&wt)[KT]) {
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int dt = 0; dt < NS; ++dt)
                    acc[dt] = mfma_f32(T[(16 * t + 4 * g + e) * P + DP * hl + 16 * dt + i], wt[t][e], acc[dt]);
    };
    fetch(0);
    for (int step = 0; step < 2 * nblocks; ++step) {
        const int sweep = step >= nblocks ? 1 : 0, k0 = KB * (step - sweep * nblocks);
        if (step) __syncthreads();               // the previous block has been read
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tid + 256 * u;
            *(f32x4 *)(Ks + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(kr[u], idx % (CW / 4), hg * HPW, D);
            *(f32x4 *)(Vs + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(vr[u], idx % (CW / 4), hg * HPW, D);
        }
        __syncthreads();
        if (nblocks > 1 && step + 1 < 2 * nblocks) fetch(KB * ((step + 1) % nblocks));
        f32x4 st[KT], dp[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) st[t] = dp[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const f32x4 kf = *(const f32x4 *)(Ks + (16 * t + i) * P + DP * hl + 16 * s + 4 * g);
                const f32x4 vf = *(const f32x4 *)(Vs + (16 * t + i) * P + DP * hl + 16 * s + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    st[t] = mfma_f32(kf[e], qf[s][e], st[t]);      // S^T[key 16 t + 4 g + j][query i]
                    dp[t] = mfma_f32(vf[e], gf[s][e], dp[t]);      // dP^T, same layout
                }
            }
        }
        const int left = kn - k0;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[t][j] = 16 * t + 4 * g + j < left ? st[t][j] : -INFINITY;
        if (sweep == 0) {
            float mx = st[0][0];
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) mx = fmaxf(mx, st[t][j]);
            const float m_new = fmaxf(m, cross_row_max(mx));          // finite: the block's first key exists
            const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c_exp);
            m = m_new;
            float ls = 0.f, ds = 0.f;
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    st[t][j] = __builtin_amdgcn_exp2f((st[t][j] - m_new) * c_exp);
                    ls += st[t][j];
                    ds = fmaf(st[t][j], dp[t][j], ds);
                }
            l = fmaf(l, alpha, cross_row_sum(ls));
            dd = fmaf(dd, alpha, cross_row_sum(ds));
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) acc[dt] *= alpha;
            contract(Vs, st);
            if (step + 1 < nblocks) continue;
            // end of the sweep: O and the statistics
            const float inv = 1.0f / l;
            dd *= inv;
            if (live) {
                float *orow = O + (itok + qtok) * D.C + h * D.d;
#pragma unroll
                for (int dt = 0; dt < NS; ++dt)
                    if (16 * dt + 4 * g < D.d) store4<VEC>(orow + 16 * dt + 4 * g, acc[dt] * inv, D.d - 16 * dt - 4 * g);
                if (g == 0) {
                    lse[(itok + qtok) * D.heads + h] = fmaf(m, c_exp, __builtin_amdgcn_logf(l));    // v_log_f32: log2
                    dsum[(itok + qtok) * D.heads + h] = dd;
                }
            }
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (nblocks > 1) continue;
        } else {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) st[t][j] = __builtin_amdgcn_exp2f((st[t][j] - m) * c_exp);
        }
        // st: exp(s - m); dS = st / l (dP - D)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[t][j] *= dp[t][j] - dd;
        contract(Ks, st);
        if (nblocks == 1) break;
    }
    if (live) {
        const float f = D.scale / l;
        float *qrow = dQKV + (itok + qtok) * C3 + h * D.d;
#pragma unroll
        for (int dt = 0; dt < NS; ++dt)
            if (16 * dt + 4 * g < D.d) store4<VEC>(qrow + 16 * dt + 4 * g, acc[dt] * f, D.d - 16 * dt - 4 * g);
    }
}

// ---------------------------------------------------------------------------
// Key side for (image, key region, key tile, HPW heads): wavefront w has 16 keys of one head.  The queries of
// all regions routed to this one (every routing entry that names it, in the order of the entries) form one
// list of rows; their Q, dO rows and statistics pass through LDS QB at a time, the next block being requested
// meanwhile:
//     S = Q K^T and dP = dO V^T,  P = exp2(scale log2(e) S - lse),  dS = P (dP - D)      (registers)
//     dV^T += dO^T P,  dK^T += Q^T dS                                                    (registers)
// and dK, dV are stored once: no atomic adds, no zeroed buffers, the same bits on every run.  A region that no
// query attends to gets zeros.
template <int DP, int HPW, bool VEC>
__global__ __launch_bounds__(256) void k_attn_bwd_kv(const float *__restrict__ QKV, const float *__restrict__ dO,
                                                     const int32_t *__restrict__ Ir, const float *__restrict__ lse,
                                                     const float *__restrict__ dsum, float *__restrict__ dQKV, Dims D,
                                                     int hgroups, int ktiles, bool by_image, lce::AddJob<float> J, int lce_blocks)
{
    typedef AttnShape<DP, HPW> L;
    constexpr int P = L::P, QB = L::KB, CW = L::CW, QTL = QB / 16, NS = DP / 16;
    __shared__ __attribute__((aligned(16))) float lds[2 * QB * P];
    float *Qs = lds, *Gs = lds + QB * P;
    static_assert(2 * QB * P >= 25 * 64, "the pass shares the buffers");
    __shared__ __attribute__((aligned(16))) float lse_s[HPW * QB], dd_s[HPW * QB];
    __shared__ int list[bwd::kListChunk], counts[16];
    int wg, wgs;
    if (lce::block_of_pass(lce_blocks, false, wg, wgs)) {
        lce::lce_block<VEC ? 2 : 1, true, 256>(J, D, mfma::swizzled(wg, wgs), lds);
        return;
    }
    const AttnWork work = attn_work(wg, wgs, by_image, ktiles, hgroups, D.R);
    const int kt = work.tile, reg = work.region, hg = work.hg, b = work.image;
    if (b >= D.B) return;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int C3 = 3 * D.C, hl = wave / L::TPH, h = hg * HPW + hl;
    const size_t itok = (size_t)b * D.N;
    const float *img = QKV + itok * C3;
    const int slot = L::QT * kt + 16 * (wave % L::TPH) + i;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n, k_inv = 1.0f / (float)D.k;
    const int ktok = at.origin(reg) + at.slot(min(slot, D.n - 1));
    f32x4 kf[NS], vf[NS], ak[NS], av[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        kf[s] = blank_head_chunk<DP, VEC>(load_head_chunk<DP, VEC>(img + (size_t)ktok * C3 + D.C, 4 * s + g, h, D), 4 * s + g, h, D);
        vf[s] = blank_head_chunk<DP, VEC>(load_head_chunk<DP, VEC>(img + (size_t)ktok * C3 + 2 * D.C, 4 * s + g, h, D), 4 * s + g, h, D);
        ak[s] = av[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float c_exp = D.scale * 1.4426950408889634f;
    const int entries = D.R * D.k;
    const int32_t *irb = Ir + (size_t)b * entries;
    constexpr int NL = QB * CW / 4 / 256;
    static_assert(HPW * QB <= 256, "one statistics entry per thread");
    f32x4 qr[NL], gr[NL];
    float next_lse = INFINITY, next_dd = 0.f;
    for (int e0 = 0; e0 < entries; e0 += bwd::kListChunk) {
        const int rows = bwd::collect_entries(irb, entries, e0, reg, D.R, list, counts) * D.n;
        auto query_token = [&](int row) {
            const int e = divide(row, D.n, n_inv);
            return at.origin(divide(list[e], D.k, k_inv)) + at.slot(row - e * D.n);
        };
        auto fetch = [&](int r0) {
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const int idx = tid + 256 * u;
                const int tok = query_token(min(r0 + idx / (CW / 4), rows - 1));      // past the end: weight zero, see below
                qr[u] = load_head_chunk<DP, VEC>(img + (size_t)tok * C3, idx % (CW / 4), hg * HPW, D);
                gr[u] = load_head_chunk<DP, VEC>(dO + (itok + tok) * D.C, idx % (CW / 4), hg * HPW, D);
            }
            if (tid < HPW * QB) {
                const int row = r0 + tid % QB, hh = hg * HPW + tid / QB;
                const bool ok = row < rows && hh < D.heads;
                const size_t at = ok ? (itok + query_token(row)) * D.heads + hh : 0;
                next_lse = ok ? lse[at] : INFINITY;                // a missing row: P = exp2(-inf) = 0
                next_dd = ok ? dsum[at] : 0.f;
            }
        };
        if (rows > 0) fetch(0);
        for (int r0 = 0; r0 < rows; r0 += QB) {
            __syncthreads();                     // the previous block has been read
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const int idx = tid + 256 * u;
                *(f32x4 *)(Qs + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(qr[u], idx % (CW / 4), hg * HPW, D);
                *(f32x4 *)(Gs + (idx / (CW / 4)) * P + 4 * (idx % (CW / 4))) = blank_head_chunk<DP, VEC>(gr[u], idx % (CW / 4), hg * HPW, D);
            }
            if (tid < HPW * QB) {
                lse_s[tid] = next_lse;
                dd_s[tid] = next_dd;
            }
            __syncthreads();
            if (r0 + QB < rows) fetch(r0 + QB);
            const int tiles = (min(QB, rows - r0) + 15) / 16;
#pragma unroll
            for (int t = 0; t < QTL; ++t) {
                if (t >= tiles) break;
                f32x4 st = {0.f, 0.f, 0.f, 0.f}, dp = st;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const f32x4 qv = *(const f32x4 *)(Qs + (16 * t + i) * P + DP * hl + 16 * s + 4 * g);
                    const f32x4 gv = *(const f32x4 *)(Gs + (16 * t + i) * P + DP * hl + 16 * s + 4 * g);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        st = mfma_f32(qv[e], kf[s][e], st);       // S[query 16 t + 4 g + j][key i]
                        dp = mfma_f32(gv[e], vf[s][e], dp);
                    }
                }
                const f32x4 l4 = *(const f32x4 *)(lse_s + hl * QB + 16 * t + 4 * g);
                const f32x4 d4 = *(const f32x4 *)(dd_s + hl * QB + 16 * t + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(st[e], c_exp, -l4[e])), ds = p * (dp[e] - d4[e]);
#pragma unroll
                    for (int dt = 0; dt < NS; ++dt) {
                        const int at = (16 * t + 4 * g + e) * P + DP * hl + 16 * dt + i;
                        av[dt] = mfma_f32(Gs[at], p, av[dt]);     // dV^T[channel 16 dt + 4 g + j][key i]
                        ak[dt] = mfma_f32(Qs[at], ds, ak[dt]);
                    }
                }
            }
        }
    }
    if (slot < D.n && h < D.heads) {
        float *row = dQKV + (itok + ktok) * C3 + h * D.d;
#pragma unroll
        for (int dt = 0; dt < NS; ++dt) {
            const int ch = 16 * dt + 4 * g;
            if (ch >= D.d) continue;
            store4<VEC>(row + D.C + ch, ak[dt] * D.scale, D.d - ch);
            store4<VEC>(row + 2 * D.C + ch, av[dt] + load4<VEC>(row + 2 * D.C + ch, D.d - ch), D.d - ch);    // LCE^T(dO) is there
        }
    }
}

// ---------------------------------------------------------------------------
// Part[share][a][n] = sum over the share's tokens t of A[t][a] B[t][n]: the weight gradients, contractions over
// all tokens.  A 64 x 64 block of the output per workgroup, both operands staged 32 tokens at a time (the next
// 32 requested meanwhile) and read as 16 consecutive channels of 4 token rows; the wavefronts split the block
// 2 x 2.  Two such products per launch.
template <typename TA, typename TB>
struct TnJob {
    const TA *A;
    const TB *Bm;
    float *Part;
    int lda, ldb, KA, N;
    __host__ __device__ int blocks() const { return ((N + 63) / 64) * ((KA + 63) / 64); }      // of a share
};

template <bool VEC, typename TA, typename TB>
__device__ __forceinline__ void tn_tile(const TnJob<TA, TB> &J, int block, int share, long M, int share_tokens, float *smem)
{
    constexpr int P = 64 + 4, TT = 32, NL = TT * 16 / 256;
    float *As = smem, *Bs = smem + TT * P;
    const int nb = (J.N + 63) / 64, n0 = 64 * (block % nb), a0 = 64 * (block / nb);
    const long t_begin = (long)share * share_tokens, t_end = min(M, t_begin + share_tokens);
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    f32x4 ra[NL], rb[NL], acc[2][2];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u / 2][u % 2] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](long t0) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tid + 256 * u, c = 4 * (idx % 16);
            const long tc = min(t0 + idx / 16, t_end - 1);
            ra[u] = load4<VEC>(J.A + tc * J.lda + (VEC ? min(a0 + c, J.KA - 4) : a0 + c), J.KA - a0 - c);
            rb[u] = load4<VEC>(J.Bm + tc * J.ldb + (VEC ? min(n0 + c, J.N - 4) : n0 + c), J.N - n0 - c);
        }
    };
    fetch(t_begin);
    for (long t0 = t_begin; t0 < t_end; t0 += TT) {
        if (t0 > t_begin) __syncthreads();
        if (t0 + TT > t_end) {               // blanked here, not behind the loads: the prefetch stays in flight
#pragma unroll
            for (int u = 0; u < NL; ++u)
                if (t0 + (tid + 256 * u) / 16 >= t_end) ra[u] = rb[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tid + 256 * u;
            *(f32x4 *)(As + (idx / 16) * P + 4 * (idx % 16)) = ra[u];
            *(f32x4 *)(Bs + (idx / 16) * P + 4 * (idx % 16)) = rb[u];
        }
        __syncthreads();
        if (t0 + TT < t_end) fetch(t0 + TT);
#pragma unroll
        for (int s = 0; s < TT / 4; ++s) {
            float a[2], bv[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                a[u] = As[(4 * s + g) * P + 32 * (wave / 2) + 16 * u + i];
                bv[u] = Bs[(4 * s + g) * P + 32 * (wave % 2) + 16 * u + i];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v) acc[u][v] = mfma_f32(a[u], bv[v], acc[u][v]);
        }
    }
    float *out = J.Part + (size_t)share * J.KA * J.N;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = a0 + 32 * (wave / 2) + 16 * u + 4 * g + j, n = n0 + 32 * (wave % 2) + 16 * v + i;
                if (a < J.KA && n < J.N) out[(size_t)a * J.N + n] = acc[u][v][j];
            }
}

// What is left once dQ, dK and dV are there, in one launch: dX = [dQ | dK | dV] Wqkv^T (J), dWqkv and dWo (J0, J1).
// SPLIT: J by split_tile, float32.
template <bool VEC, int BN, typename T, bool SPLIT = false>
__global__ __launch_bounds__(256) void k_gemm_end(TnJob<T, float> J0, TnJob<float, T> J1, long M, int share_tokens, int tn_blocks, GemmJob<float, T, T> J)
{
    constexpr size_t n = gemm_lds_floats<BN, true>(), tn = 2 * 32 * (64 + 4);
    __shared__ __attribute__((aligned(16))) float smem[n > tn ? n : tn];
    const int block = (int)blockIdx.x - tn_blocks;
    if (block >= 0) {
        if constexpr (SPLIT) {
            static_assert(split_lds_floats<1, 4>() <= n, "the sums fit");
            split_tile<true, 1, 4>(J, block, smem);
            return;
        }
        any_gemm_tile<true, VEC, BN>(J, block, (int)gridDim.x - tn_blocks, smem);
        return;
    }
    // the blocks of a share one after the other, so that an XCD's L2 has its tokens
    const int at = mfma::swizzled(blockIdx.x, tn_blocks), each = J0.blocks() + J1.blocks(), share = at / each, rest = at - share * each;
    if ((long)share * share_tokens >= M) return;
    if (rest < J0.blocks()) tn_tile<VEC>(J0, rest, share, M, share_tokens, smem);
    else tn_tile<VEC>(J1, rest - J0.blocks(), share, M, share_tokens, smem);
}

}  // namespace f32
}  // namespace bra
