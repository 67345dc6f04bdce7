// Matrix-core pipeline for the shapes that the specialised kernels do not take: any C that is
// a multiple of 64, heads of 32 or 64 channels, any region size and count, e.g. the last stage
// of the paper's backbones (7x7 map, S = 7: one token per region, k = S^2, C = 512), the wider
// variants' stages (C = 384, 768), S = 16 on large maps, and the plain-ViT adaptation of the
// appendix (32x32 map, S = 8, k = 12, 12 heads of 64 channels).
//
//   k_gemm_means  Q | K | V = X Wqkv (Eq. 3), bf16 out, and Q^r | K^r, the means of Q and K over each region, from the
//                 float32 results (Sec. 3.2)
//   or, on larger maps (means_from_projection), k_pool_wide, Xr[b, r, :] = mean of the region's tokens, float32, and k_gemm_dma with
//                 Q^r | K^r = Xr [Wq | Wk] in the launch of Q | K | V: the means are split exactly into three bf16 terms, so
//                 the products are those of the float32 computation
//                 (one token per region: no means, the token projection leaves float32 copies of Q and K instead)
//   k_route_lce   rows of A^r = Q^r (K^r)^T (Eq. 4) and their top-k (Eq. 5), and LCE(V) (Eq. 7) in float32 beside them
//   k_attn_rows (regions of up to 32 tokens) or k_attn_gen, O = the two together   (Eq. 6)
//   or, on large maps, k_route_rows, the attention and k_lce_add
//   or k_route_rows and the image-resident attention with its own LCE (map_tail_pays; bra_mfma_small.hip)
//   k_gemm_dma    Y = O Wo (Eq. 2), or with two heads and regions of more than 32 tokens in k_attn_gen
#include "bra_attn_dev.h"
#include "bra_gemm.h"
#include "bra_lce_dev.h"

#include <stdlib.h>

namespace bra {

using namespace mfma;

namespace {

// SUB (a power of two up to 32) consecutive lanes share one (image, region, 8-channel chunk): lane s adds
// tokens s, s + SUB, .. of the region (row-major), then the partial sums are combined pairwise
// in a fixed order.
// PAD: X is the caller's map of pad.H x pad.W tokens, zero beyond.
template <bool PAD>
__global__ __launch_bounds__(256) void k_pool_wide(const bf16_t *__restrict__ X, float *__restrict__ Xr, Dims D,
                                                   int SUB, GemmRows pad)
{
    const int CH = D.C / 8;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const long item = idx / SUB;
    const int sub = (int)(idx % SUB);
    const bool valid = item < (long)D.B * D.R * CH;
    const long it = valid ? item : 0;
    const int cc = (int)(it % CH), r = (int)((it / CH) % D.R), b = (int)(it / ((long)CH * D.R));
    const int H = PAD ? pad.H : D.H, W = PAD ? pad.W : D.W, y0 = (r / D.S) * D.rh, x0 = (r % D.S) * D.rw;
    const bf16_t *base = X + (((size_t)b * H + y0) * W + x0) * D.C + cc * 8;
    const float rw_inv = 1.0f / (float)D.rw;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int slot = sub; slot < D.n; slot += SUB) {
        const int y = fast_div(slot, rw_inv), x = slot - y * D.rw;
        const bool in = !PAD || (y0 + y < H && x0 + x < W);
        u32x4 v = *(const u32x4 *)(in ? base + ((size_t)y * W + x) * D.C : X);
        if (PAD && !in) v = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[2 * e] += bf16_lo(v[e]);
            acc[2 * e + 1] += bf16_hi(v[e]);
        }
    }
    for (int off = 1; off < SUB; off *= 2)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off);
    if (valid && sub == 0) {
        float *dst = Xr + ((size_t)b * D.R + r) * D.C + cc * 8;
        const float inv = 1.0f / (float)D.n;
        *(f32x4 *)dst = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
        *(f32x4 *)(dst + 4) = f32x4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
    }
}

// What an output is added to (LCE(V), float32 with the upper halves of the bits in O and the lower ones in Low: the sum rounds
// once): the lane's four channels of 16-channel tile dt of NQ query tiles.
template <int NQ, int NDT>
struct Added {
    u32x2 hi[NQ][NDT], lo[NQ][NDT];

    __device__ __forceinline__ void load(const bf16_t *O, const bf16_t *Low, const size_t (&token)[NQ], int C, int g)
    {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                hi[q][dt] = *(const u32x2 *)(O + token[q] * C + 16 * dt + 4 * g);
                lo[q][dt] = *(const u32x2 *)(Low + token[q] * C + 16 * dt + 4 * g);
            }
    }
    __device__ __forceinline__ f32x4 to(f32x4 x, int q, int dt) const
    {
        const u32x2 h = hi[q][dt], l = lo[q][dt];
        return x + __builtin_bit_cast(f32x4, u32x4{pair_lo(l[0], h[0]), pair_hi(l[0], h[0]), pair_lo(l[1], h[1]), pair_hi(l[1], h[1])});
    }
};

// ---------------------------------------------------------------------------
// Routed attention (Eq. 6, Eq. 1) for any region size and heads of 32 or 64 channels.  Q comes multiplied by
// scale * log2(e), so scores are exponents of 2.
//
// Regions of more than 32 tokens: workgroup (image, group of 64 channels = 2 or 1 heads, region, tile of 64 NQ queries of the
// region), a wavefront with NQ query tiles of 16 and HPW heads.  The k n routed keys are taken 64 at a time: their K and V rows (the
// group's 128 bytes each, found by index in the projected maps) go straight from memory into one of two LDS buffers while
// the other is worked on; 16-byte pieces are exchanged (piece c of row r at c ^ r % 8), so that K's row reads and V's
// transposing reads meet different banks.  Queries past the end of the region and keys past k n
// repeat the last one and are masked.
// Bound by vector issue: 2 x 208 x 304 x 64, 16 x 16 regions, k = 4 (250 M scores) takes 64 us, the convolution it is added to
// with it.  A wavefront's 16 x 64 scores take 16 2^x (8 clocks each), 15 additions, 8 conversions, about 6 other vector instructions
// and 8 products, of which each keeps the vector pipe for about 9 clocks beside 2^x.  One head per wavefront and eight of
// them, 124 registers: four wavefronts per SIMD where both heads (154 registers) left three and the last quarter of 1024 workgroups
// to a second round (70.7 us); four registers of -m as the products' accumulator input instead of moves for every tile.  One
// query tile per wavefront instead of two: 8 us more (4 x 64 x 64 x 384, heads of 64, k = 4: 45 for 39).
template <int HD, int HPW>
constexpr int genWaves = 4 * (64 / HD) / HPW;

// With OUT also Y = O Wo (Eq. 7), where C is the 64 channels of the workgroup: a lane's channels of an output are the operand of that product as they
// are, Wo lies in LDS as a block of V does; O is not written.  Y may be where Low is: a workgroup reads its tokens before it writes them.
// A launch and two passes over O less: padded 2 x 200 x 300, S = 16, k = 4 107.7 -> 102.5 us, 1 x 200 x 300, k = 2 56.1 -> 50.9, 1 x 100 x 150, k = 8
// 41.3 -> 38.7; 4 x 112 x 112, S = 16, k = 4 43.9 -> 42.4.
struct OutMap {
    const bf16_t *Wo;
    bf16_t *Y;
    int H, W;                // of Y, where D describes a padded map, else 0
};

template <int HD, int NQ, int HPW, bool WALK, bool OUT>
__global__ __launch_bounds__((64 * genWaves<HD, HPW>), HD == 32 && HPW == 1 ? 4 : 3) void k_attn_gen(AttnArgs A, bf16_t *O, Dims D, int qtiles, const bf16_t *Low, OutMap out)
{
    static_assert(!OUT || HD == 32, "two heads");
    constexpr int WAVES = genWaves<HD, HPW>, PARTS = WAVES / 4, KSD = HD / 32, NDT = HD / 16;
    __shared__ __attribute__((aligned(16))) bf16_t K0[64 * 64];
    __shared__ __attribute__((aligned(16))) bf16_t K1[64 * 64];
    __shared__ __attribute__((aligned(16))) bf16_t V0[64 * 64];
    __shared__ __attribute__((aligned(16))) bf16_t V1[64 * 64];
    __shared__ __attribute__((aligned(16))) bf16_t Ws[OUT ? 64 * 64 : 8];
    extern __shared__ int origins[];             // [k]: first token of the routed regions; with WALK [n]: tokens of a region's slots
    const int C = D.C, ncg = C / 64, n = D.n, kn = D.kn;
    // workgroups of an image and channel group share an L2: a gathered row of 128 bytes is a line of one group (10 x 64 x 64 x 384,
    // k = 6: layer 153.8 us; groups next to each other 158.0, all over the XCDs 160.1)
    const int block = swizzled_block();
    const int qt = block % qtiles, reg = (block / qtiles) % D.R;
    const int cg = (block / (qtiles * D.R)) % ncg, b = block / (qtiles * D.R * ncg);
    if (b >= D.B) return;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), part = wave % PARTS, qw = wave / PARTS, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const float rw_inv = 1.0f / (float)D.rw, n_inv = 1.0f / (float)n, s_inv = 1.0f / (float)D.S;
    const size_t img = (size_t)b * D.N * C + 64 * cg;
    const int c0 = 64 / PARTS * part;             // the wavefront's first channel of the group
    auto region_origin = [&](int r) {
        const int ry = fast_div(r, s_inv);
        return ry * D.rh * D.W + (r - ry * D.S) * D.rw;
    };
    auto in_region = [&](int slot) {
        const int sy = fast_div(slot, rw_inv);
        return sy * D.W + slot - sy * D.rw;
    };
    size_t qtok[NQ];
    bf16x8 qf[NQ][HPW][KSD];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        qtok[q] = (size_t)region_origin(reg) + in_region(min(64 * NQ * qt + 16 * (NQ * qw + q) + i, n - 1));
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks)
                qf[q][hh][ks] = *(const bf16x8 *)(A.Q + img + qtok[q] * C + c0 + HD * hh + 32 * ks + 8 * g);
    }
    Added<NQ, NDT * HPW> added;
    if (NQ == 1 && Low) added.load(O + img + c0, Low + img + c0, qtok, C, g);
    const int32_t *irp = A.Ir_src + ((size_t)b * D.R + reg) * D.k;
    const bool report = A.Ir_out && A.Ir_out != A.Ir_src && qt == 0 && cg == 0;
    for (int p = tid; p < D.k; p += 64 * WAVES) {
        const int j = irp[p];
        origins[p] = region_origin(region_index(j, D.R));
        if (report) A.Ir_out[((size_t)b * D.R + reg) * D.k + p] = j;
    }
    int *slots = origins + D.k;
    if (WALK)
        for (int t = tid; t < n; t += 64 * WAVES) slots[t] = in_region(t);
    // the operands have arrived before the loop: otherwise the compiler waits for them, and with them for the direct loads
    // in flight, in every pass
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) asm volatile("" : "+v"(qf[q][hh][ks]));
    // direct loads: a wavefront brings its share of the rows of K and V, 8 rows of 8 pieces each, block after block
    constexpr int LOADS = 8 / WAVES;
    RowWalk<LOADS> walk;
    if constexpr (WALK) walk.start(8 * LOADS * wave + lane / 8, 8, 64, n, n_inv);
    const unsigned piece = 16 * ((lane % 8) ^ (lane / 8));
    auto request = [&](int k0, unsigned Ks, unsigned Vs) {
        lds_reads_done();
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const unsigned at = 1024 * (LOADS * wave + u);
            if constexpr (WALK) {
                const unsigned off = row_offset(walk.token(u, origins, D.k - 1, slots), C, piece);
                load_to_lds_untracked(A.K + img, off, Ks + at);
                load_to_lds_untracked(A.V + img, off, Vs + at);
            } else {
                const int key = min(k0 + 8 * (LOADS * wave + u) + lane / 8, kn - 1), p = fast_div(key, n_inv);
                const size_t e = img + (size_t)(origins[p] + in_region(key - p * n)) * C + piece / 2;
                load_to_lds_untracked(A.K + e, Ks + at);
                load_to_lds_untracked(A.V + e, Vs + at);
            }
        }
        if constexpr (WALK) walk.advance();
    };
    constexpr bool KEPT = HD == 32 && HPW == 1;      // registers for four copies of -m
    float m[NQ][HPW], l[NQ][HPW];
    f32x4 acc[NQ][HPW][NDT], neg[NQ][HPW];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            m[q][hh] = l[q][hh] = 0.f;
            neg[q][hh] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) acc[q][hh][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto block_of_keys = [&](int k0, const bf16_t *Ks, const bf16_t *Vs, auto first) {
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            bf16x8 pb[NQ][2];
            {
                bf16x8 kf[4][KSD];
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int ks = 0; ks < KSD; ++ks) kf[t][ks] = row_operand(Ks, 16 * t + i, (c0 + HD * hh) / 8 + 4 * ks + g);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    f32x4 s[4];
                    const float was = m[q][hh];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float neg1 = -m[q][hh];
                        s[t] = KEPT ? neg[q][hh] : f32x4{neg1, neg1, neg1, neg1};
#pragma unroll
                        for (int ks = 0; ks < KSD; ++ks) s[t] = mfma16(kf[t][ks], qf[q][hh][ks], s[t]);
                    }
                    if (k0 + 64 > kn) {
#pragma unroll
                        for (int t = 0; t < 4; ++t)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                if (k0 + 16 * t + 4 * g + j >= kn) s[t][j] = -INFINITY;
                    }
                    softmax_step<decltype(first)::value>(s, m[q][hh], l[q][hh], acc[q][hh], pb[q]);
                    if (KEPT && (decltype(first)::value || __builtin_amdgcn_ballot_w64(m[q][hh] != was) != 0)) {
                        const float neg1 = -m[q][hh];
                        neg[q][hh] = f32x4{neg1, neg1, neg1, neg1};
                        asm volatile("" : "+v"(neg[q][hh]));      // four registers: made anew from one, they are 3 moves per product
                    }
                    if (NQ > 1) __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const bf16x8 vf = column_operand(Vs, 32 * tp, c0 + HD * hh + 16 * dt, g, i);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) acc[q][hh][dt] = mfma16(vf, pb[q][tp], acc[q][hh][dt]);
                }
            __builtin_amdgcn_sched_barrier(0);    // one head at a time: interleaved, they take twice the registers
        }
    };
    const bool idle = 64 * NQ * qt + 16 * NQ * qw >= n;      // a wavefront without queries only brings its rows
    __syncthreads();                              // the table is in place
    if constexpr (OUT)
#pragma unroll
        for (int u = 0; u < LOADS; ++u)
            load_to_lds_untracked(out.Wo + 64 * (8 * (LOADS * wave + u) + lane / 8) + piece / 2, lds_address(Ws) + 1024 * (LOADS * wave + u));
    const unsigned kv[2][2] = {{lds_address(K0), lds_address(V0)}, {lds_address(K1), lds_address(V1)}};
    request(0, kv[0][0], kv[0][1]);
    arrive_barrier();
    if (64 < kn) request(64, kv[1][0], kv[1][1]);
    if (!idle) block_of_keys(0, K0, V0, std::true_type{});
    for (int k0 = 64; k0 < kn; k0 += 128) {
        arrive_barrier();
        if (k0 + 64 < kn) request(k0 + 64, kv[0][0], kv[0][1]);
        if (!idle) block_of_keys(k0, K1, V1, std::false_type{});
        if (k0 + 64 >= kn) break;
        arrive_barrier();
        if (k0 + 128 < kn) request(k0 + 128, kv[1][0], kv[1][1]);
        if (!idle) block_of_keys(k0 + 64, K0, V0, std::false_type{});
    }
    if (NQ > 1 && Low) added.load(O + img + c0, Low + img + c0, qtok, C, g);      // registers that the sweep does not have
    if constexpr (OUT) {
        bf16x8 o[NQ][2];                         // operands: slot e of head h is channel 32 h + 16 (e / 4) + 4 g + e % 4
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                const float inv = 1.0f / cross_row_sum(l[q][hh]);
                const f32x4 v0 = added.to(acc[q][hh][0] * inv, q, NDT * hh), v1 = added.to(acc[q][hh][1] * inv, q, NDT * hh + 1);
                const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                o[q][hh] = pack8(v);
            }
        if constexpr (PARTS == 2) {              // the heads' wavefronts of the same queries exchange them, each forms half of Y's columns
            __syncthreads();                     // the last block has been read
#pragma unroll
            for (int q = 0; q < NQ; ++q) *(bf16x8 *)((q ? K1 : K0) + 512 * (2 * qw + part) + 8 * lane) = o[q][0];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) o[q][hh] = *(const bf16x8 *)((q ? K1 : K0) + 512 * (2 * qw + hh) + 8 * lane);
        } else {
            __syncthreads();                     // Low of all queries has been read
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int slot = 64 * NQ * qt + 16 * (NQ * qw + q) + i, sy = fast_div(slot, rw_inv), ry = fast_div(reg, s_inv);
            const int y = ry * D.rh + sy, x = (reg - ry * D.S) * D.rw + slot - sy * D.rw;
            const int H = out.H ? out.H : D.H, W = out.H ? out.W : D.W;
            const bool store = slot < n && y < H && x < W;
            bf16_t *to = out.Y + (((size_t)b * H + y) * W + x) * 64 + 4 * g;
#pragma unroll
            for (int u = 0; u < 4 / PARTS; ++u) {
                const int t = 4 / PARTS * part + u;
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) v = mfma16(column_operand(Ws, 32 * hh, 16 * t, g, i), o[q][hh], v);
                if (store) *(u32x2 *)(to + 16 * t) = pack4(v);
            }
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const bool store = 64 * NQ * qt + 16 * (NQ * qw + q) + i < n;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            const float inv = 1.0f / cross_row_sum(l[q][hh]);
            if (!store) continue;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                f32x4 v = acc[q][hh][dt] * inv;
                if (Low) v = added.to(v, q, NDT * hh + dt);
                *(u32x2 *)(O + img + qtok[q] * C + c0 + HD * hh + 16 * dt + 4 * g) = pack4(v);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The same for regions of at most 32 tokens (16 NQ of them in NQ query tiles), where the tile of 64 queries above leaves
// half or more of its wavefronts with copies: a wavefront works on its own, with all queries of a region and 64 channels
// (2 or 1 heads), any four of them in a workgroup.  It brings its K and V rows straight from memory into its own part of LDS, 32 keys at a time;
// a block's operands go to registers, and the block that takes its place is requested before it is worked on (with two buffers: the other one).  There is no barrier.  Rows of 128
// bytes lie unpadded, their pieces exchanged as above.
// Bound by the gather out of the L2s: 302 MB for 8 images of 32 x 32 x 768 with 12 regions of 16 tokens each; with few keys by
// the chain of loads before the first product (routing entry, row, output) and the wavefronts that hide it, so that what the output is added to
// and the queries are requested with the routing entries (64 x 16 x 24 x 384, k = 1: attention 51.7 -> 31.9 us, layer 146 ->
// 126; 32 x 16 x 16 x 768, k = 2: 49.1 -> 29.7; 29 x 8 x 8 x 768, k = 33: 46.1 -> 40.3).
// One buffer of 32 keys, so that four workgroups share a compute unit, where there are wavefronts for it; two, one ahead, where two per unit
// take them all (kRowsShared) or registers leave no room for more (NQ = 2).  Layer, two buffers / one (us): 8 x 32 x 32 x 768, k = 12
// 97.4 / 94.6, 4 images of 24 heads 62.6 / 60.5, 16 x 21 x 21 x 512, k = 20 72.8 / 67.0, 32 x 14 x 28 x 512, k = 6 98.3 / 93.8, 8 x 28 x 28 x 384, k = 9
// 43.0 / 41.0; few: 2 x 32 x 32 x 768, k = 12 (1536 wavefronts) 45.6 / 45.9, 3 x 28 x 28 x 768, k = 6 44.0 / 44.3.
constexpr int kRowsShared = 2048;
constexpr int kRowsBuffer = 4 * 2 * 32 * 64 * 2;       // bytes

template <int HD, int NQ, int BUFFERS>
__global__ __launch_bounds__(256, NQ == 2 || BUFFERS == 2 ? 2 : 4) void k_attn_rows(AttnArgs A, bf16_t *__restrict__ O, Dims D, int items, const bf16_t *__restrict__ Low)
{
    constexpr int HPW = 64 / HD, KSD = HD / 32, NDT = HD / 16, KB = 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *S = (bf16_t *)smem;      // [buffer][wavefront][K, V][32 keys][64]
    int *origin_tables = (int *)(smem + BUFFERS * kRowsBuffer);      // [4][k]: first token of the routed regions; [4][32]: tokens of a region's slots
    const int C = D.C, ncg = C / 64, n = D.n, kn = D.kn;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, g = lane / 16, i = lane % 16;
    const int item = __builtin_amdgcn_readfirstlane(4 * swizzled_block() + wave);      // those of an image share an L2
    if (item >= items) return;
    const int cg = item % ncg, reg = (item / ncg) % D.R, b = item / (ncg * D.R);
    int *origins = origin_tables + wave * D.k, *slots = origin_tables + 4 * D.k + 32 * wave;
    const float rw_inv = 1.0f / (float)D.rw, n_inv = 1.0f / (float)n, s_inv = 1.0f / (float)D.S;
    auto region_origin = [&](int r) {
        const int ry = fast_div(r, s_inv);
        return ry * D.rh * D.W + (r - ry * D.S) * D.rw;
    };
    auto in_region = [&](int slot) {
        const int sy = fast_div(slot, rw_inv);
        return sy * D.W + slot - sy * D.rw;
    };
    const size_t img = (size_t)b * D.N * C + 64 * cg;
    const int origin = region_origin(reg);
    size_t qtok[NQ];
    bf16x8 qf[NQ][HPW][KSD];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        qtok[q] = (size_t)origin + in_region(min(16 * q + i, n - 1));
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks)
                qf[q][hh][ks] = *(const bf16x8 *)(A.Q + img + qtok[q] * C + HD * hh + 32 * ks + 8 * g);
    }
    Added<NQ, 4> added;
    if (Low) added.load(O + img, Low + img, qtok, C, g);
    const int32_t *irp = A.Ir_src + ((size_t)b * D.R + reg) * D.k;
    const bool report = A.Ir_out && A.Ir_out != A.Ir_src && cg == 0;
    for (int p = lane; p < D.k; p += kWave) {
        const int j = irp[p];
        origins[p] = region_origin(region_index(j, D.R));
        if (report) A.Ir_out[((size_t)b * D.R + reg) * D.k + p] = j;
    }
    if (lane < n) slots[lane] = in_region(lane);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the tables are read by other lanes
    // the operands have arrived before the loop: otherwise the compiler waits for them, and with them for the direct loads
    // in flight, in every pass
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) asm volatile("" : "+v"(qf[q][hh][ks]));
    // direct loads: 8 rows of 8 pieces each, block after block
    RowWalk<KB / 8> walk;
    walk.start(lane / 8, 8, KB, n, n_inv);
    const unsigned piece = 16 * ((lane % 8) ^ (lane / 8)), mine = lds_address(S + wave * 2 * KB * 64);
    auto request = [&](int at) {
        lds_reads_done();
#pragma unroll
        for (int u = 0; u < KB / 8; ++u) {
            const unsigned off = row_offset(walk.token(u, origins, D.k - 1, slots), C, piece);
            load_to_lds_untracked(A.K + img, off, mine + at + 1024 * u);
            load_to_lds_untracked(A.V + img, off, mine + at + KB * 128 + 1024 * u);
        }
        walk.advance();
    };
    float m[NQ][HPW], l[NQ][HPW];
    f32x4 acc[NQ][HPW][NDT];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            m[q][hh] = l[q][hh] = 0.f;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) acc[q][hh][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto read = [&](int buffer, int hh, bf16x8 (&kf)[2][KSD], bf16x8 (&vf)[NDT]) {
        const bf16_t *Ks = S + buffer * (kRowsBuffer / 2) + wave * 2 * KB * 64, *Vs = Ks + KB * 64;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) kf[t][ks] = row_operand(Ks, 16 * t + i, HD / 8 * hh + 4 * ks + g);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) vf[dt] = column_operand(Vs, 0, HD * hh + 16 * dt, g, i);
    };
    auto work = [&](int k0, int hh, const bf16x8 (&kf)[2][KSD], const bf16x8 (&vf)[NDT], auto first) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            f32x4 s[2];
            const float neg = -m[q][hh];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                s[t] = f32x4{neg, neg, neg, neg};
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) s[t] = mfma16(kf[t][ks], qf[q][hh][ks], s[t]);   // S^T[key 16 t + 4 g + j][query i]
            }
            if (k0 + KB > kn) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k0 + 16 * t + 4 * g + j >= kn) s[t][j] = -INFINITY;
            }
            bf16x8 pb[1];
            softmax_step<decltype(first)::value>(s, m[q][hh], l[q][hh], acc[q][hh], pb);
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) acc[q][hh][dt] = mfma16(vf[dt], pb[0], acc[q][hh][dt]);
        }
    };
    request(0);
    if constexpr (BUFFERS == 1) {
        auto block = [&](int k0, auto first) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            bf16x8 kf[HPW][2][KSD], vf[HPW][NDT];
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) read(0, hh, kf[hh], vf[hh]);
            if (k0 + KB < kn) request(0);
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) work(k0, hh, kf[hh], vf[hh], first);
        };
        block(0, std::true_type{});
        for (int k0 = KB; k0 < kn; k0 += KB) block(k0, std::false_type{});
    } else {
        // requests the keys behind the block, if there are any, and waits for the 8 loads of the block itself
        auto block = [&](int k0, int buffer, auto first) {
            if (k0 + KB < kn) {
                request((buffer ^ 1) * kRowsBuffer);
                asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                bf16x8 kf[2][KSD], vf[NDT];
                read(buffer, hh, kf, vf);
                work(k0, hh, kf, vf, first);
            }
        };
        block(0, 0, std::true_type{});
        for (int k0 = KB; k0 < kn; k0 += 2 * KB) {
            block(k0, 1, std::false_type{});
            if (k0 + KB >= kn) break;
            block(k0 + KB, 0, std::false_type{});
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const bool store = 16 * q + i < n;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            const float inv = 1.0f / cross_row_sum(l[q][hh]);
            if (!store) continue;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                f32x4 v = acc[q][hh][dt] * inv;
                if (Low) v = added.to(v, q, NDT * hh + dt);
                *(u32x2 *)(O + img + qtok[q] * C + HD * hh + 16 * dt + 4 * g) = pack4(v);
            }
        }
    }
}

struct WideWs {
    bf16_t *q, *k, *v, *o;
    float *xr, *qr, *kr;
    int32_t *ir;
    size_t bytes;
};

bool many_regions(const Dims &D) { return D.S > kFastRouteMaxS; }

bool means_from_projection(const Dims &D);

WideWs carve(const Dims &D, void *ws)
{
    WideWs w;
    char *p = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *q = p ? p + off : nullptr; off += align256(bytes); return q; };
    const size_t tok = (size_t)D.B * D.N, reg = (size_t)D.B * D.R;
    w.q = (bf16_t *)take(tok * D.C * 2);
    w.k = (bf16_t *)take(tok * D.C * 2);
    w.v = (bf16_t *)take(tok * D.C * 2);
    w.o = (bf16_t *)take(tok * D.C * 2);
    w.xr = (float *)take(means_from_projection(D) ? 0 : reg * D.C * 4);       // means of X are taken only without those of Q and K
    w.qr = (float *)take(reg * D.C * 4);
    w.kr = (float *)take(reg * D.C * 4);
    w.ir = (int32_t *)take(reg * D.k * 4);
    w.bytes = off;
    return w;
}

void launch_pool(const Dims &D, const bf16_t *X, const WideWs &w, const GemmRows &pad, hipStream_t st)
{
    // lanes per (region, chunk): up to 8 with two tokens each, beyond that with eight each (247 tokens per region, 8 lanes:
    // 14 us on a 2 x 208 x 304 x 64 map, a chain of 31 loads)
    int sub = 1;
    while ((sub < 8 && 2 * sub <= D.n) || (sub < 32 && 8 * sub <= D.n)) sub *= 2;
    const long items = (long)D.B * D.R * (D.C / 8) * sub;
    ProfScope ps(st, K_MFMA_POOL_QK);
    const dim3 grid((unsigned)((items + 255) / 256));
    if (pad.Hp) hipLaunchKernelGGL(k_pool_wide<true>, grid, dim3(256), 0, st, X, w.xr, D, sub, pad);
    else hipLaunchKernelGGL(k_pool_wide<false>, grid, dim3(256), 0, st, X, w.xr, D, sub, pad);
}

GemmRegions region_job(const Dims &D, const WideWs &w)
{
    return GemmRegions{w.xr, (long)D.B * D.R, 2 * D.C, {w.qr, w.kr}, D.C};
}

GemmMeans means_job(const Dims &D, const WideWs &w, int H, int W)
{
    return GemmMeans{{w.qr, w.kr}, D.B * D.R, D.R, D.S, D.n, D.rh, D.rw, H ? H : D.H, H ? W : D.W, 1.0f / D.n, 1.0f / D.R, 1.0f / D.S, 1.0f / D.rw};
}

// The means of Q and K out of the token projection's float32 results, whose tiles then go region by region, in the place of a pooling
// pass and a region-level product: always the faster for bra_forward, by 5 us (a launch) on small maps and the region-level product's
// time on larger ones.  bra_route, which has to decide on the same bits, then projects all tokens instead of their means: the
// line lies where that takes as long.  bra_route / bra_forward before -> now (us): 1 x 28 x 28 x 384, k = 9 19.0 -> 12.4 / 33.1 -> 26.7,
// 6 x 14 x 14 x 256 16.5 -> 11.2 / 27.8 -> 22.4, 64 x 14 x 14 x 384 30.7 -> 24.4 / 77.5 -> 66.7, 32 x 16 x 16 x 768 41.8 -> 36.1 / 123.5 ->
// 101.4, 4 x 32 x 32 x 384 20.2 -> 14.8 / 39.9 -> 35.8; beyond: 8 x 32 x 32 x 768 32.4 -> 38.2 / 104.5 -> 99.0, 20 x 56 x 56 x 192 18.9 -> 25.6 /
// 112.0 -> 106.6.  Regions of up to 4 tokens, whose means are a quarter of the tokens or more, at any size: 64 x 14 x 14 x 192 22.6 -> 16.1 / 51.4 -> 44.1,
// x 384 31.3 -> 26.8 / 84.4 -> 71.7, x 768 55.7 -> 51.3 / 177 -> 142, 96 x 14 x 14 x 448 48.2 -> 43.8 / 142.7 -> 121.9, 100 x 14 x 14 x 768 76.6 -> 77.3 / 272 -> 212, 150 x 14 x 14 x
// 512 68.5 -> 65.1 / 226 -> 184.  They are the more exact ones too: A^r of 64 x 14 x 14 x 384 is 1.7e-7 from float64 (2-norm, relative), with the means
// of the tokens 2.7e-7, x 192 1.4e-7 and 1.9e-7.  By millions of values and tokens per region, bra_route before -> now: 8 of C = 192 11.5 37.6 -> 37.9, of C = 384 9.6
// 32.4 -> 33.1, of C = 768 3.0 30.7 -> 25.7, 7.8 37.1 -> 41.4; 16 4.7 18.5 -> 16.7 (C = 192), 9.4 26.4 -> 30.4 (384), 7.9 32.1 -> 40.8 (768); 64 4.7
// 16.8 -> 16.8, 3.1 20.1 -> 17.0, 3.1 28.4 -> 25.5; 36, of which a tile of 64 rows leaves 28 idle, 2.0 15.8 -> 14.0, 4.7 16.7 -> 18.0 (192), 4.1 20.1 -> 22.8 (384).
bool means_from_projection(const Dims &D)
{
    if (D.n == 1 || D.n > kMeansMaxTokens) return false;
    const long values = (long)D.B * D.N * D.C;
    if (D.n <= 4) return true;
    if (D.n <= 9) return values <= (D.C <= 384 ? 8L << 20 : 11L << 19);
    if (D.n <= 16) return values <= 5L << 20;
    return values <= (D.n > 32 && D.n < 60 ? 2L << 20 : 4L << 20);
}

template <int HD, int NQ, int BUFFERS>
int launch_attn_rows_b(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, int items, hipStream_t st)
{
    const int blocks = (items + 3) / 4;
    const size_t smem = (size_t)BUFFERS * kRowsBuffer + (size_t)4 * (D.k + 32) * sizeof(int);
    static bool opted = false;
    if (!opted && smem > 64 * 1024) {
        if (hipFuncSetAttribute((const void *)k_attn_rows<HD, NQ, BUFFERS>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess) return BRA_ERR_LAUNCH;
        opted = true;
    }
    hipLaunchKernelGGL((k_attn_rows<HD, NQ, BUFFERS>), dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), smem, st, A, O, D, items, Low);
    return BRA_OK;
}

template <int HD, int NQ>
int launch_attn_rows_t(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, hipStream_t st)
{
    const int items = D.B * D.R * (D.C / 64);
    return D.kn > 32 && (NQ == 2 || items <= kRowsShared) ? launch_attn_rows_b<HD, NQ, 2>(D, A, O, Low, items, st) : launch_attn_rows_b<HD, NQ, 1>(D, A, O, Low, items, st);
}

int launch_attn_rows(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, hipStream_t st)
{
    if (D.d == 32) return D.n <= 16 ? launch_attn_rows_t<32, 1>(D, A, O, Low, st) : launch_attn_rows_t<32, 2>(D, A, O, Low, st);
    return D.n <= 16 ? launch_attn_rows_t<64, 1>(D, A, O, Low, st) : launch_attn_rows_t<64, 2>(D, A, O, Low, st);
}

template <int HD, int NQ, int HPW, bool WALK, bool OUT>
void launch_attn_gen_w(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, const OutMap &out, hipStream_t st)
{
    const int qtiles = (D.n + 64 * NQ - 1) / (64 * NQ);
    const dim3 grid((unsigned)(((long)D.B * D.R * qtiles * (D.C / 64) + 7) / 8 * 8));
    const size_t smem = (size_t)(D.k + (WALK ? D.n : 0)) * sizeof(int);
    hipLaunchKernelGGL((k_attn_gen<HD, NQ, HPW, WALK, OUT>), grid, dim3(64 * genWaves<HD, HPW>), smem, st, A, O, D, qtiles, Low, out);
}

// Rows by walking (a table of the region's tokens more, an addition instead of divisions) from more than three blocks of keys on;
// a kernel of its own for each: both ways in one take 125 registers instead of 118 and 120 (one query tile, heads of 32).  Layer,
// both in one / by divisions / by walking (us): 40 x 56 x 56 x 192, k = 1 (one block) 176.6 / 174.0 / 174.5; 30 x 42 x 42 x 192, k = 5 (180 keys)
// 114.8 / 110.3 / 113.1; 20 x 77 x 77 x 64, k = 2 (242) 73.9 / 74.4 / 73.7; 2 x 200 x 300 x 64, S = 16, k = 4 (988) 115.8 / 115.1 / 114.2.
template <int NQ, int HPW>
void launch_attn_gen_t(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, const OutMap &out, hipStream_t st)
{
    const bool walks = walk_ok(D) && D.kn > 192;
    if (out.Y) walks ? launch_attn_gen_w<32, NQ, HPW, true, true>(D, A, O, Low, out, st) : launch_attn_gen_w<32, NQ, HPW, false, true>(D, A, O, Low, out, st);
    else if (D.d == 32) walks ? launch_attn_gen_w<32, NQ, HPW, true, false>(D, A, O, Low, out, st) : launch_attn_gen_w<32, NQ, HPW, false, false>(D, A, O, Low, out, st);
    else walks ? launch_attn_gen_w<64, NQ, 1, true, false>(D, A, O, Low, out, st) : launch_attn_gen_w<64, NQ, 1, false, false>(D, A, O, Low, out, st);
}

// Low: if not NULL, the output is added to what O and it hold (LCE(V)).  out.Y: not NULL for the output projection as well (C = 64, heads of 32, Low).
void launch_attn_gen(const Dims &D, const AttnArgs &A, bf16_t *O, const bf16_t *Low, const OutMap &out, hipStream_t st)
{
    // two query tiles per wavefront (every K and V operand read serves both; measured above) where the wider tile leaves no
    // more than an eighth of its queries empty beyond the narrow one and there are workgroups enough.  Both heads in a wavefront where a
    // prologue paid by half as many outweighs the fourth wavefront per SIMD: two query tiles and many workgroups with few keys (layer, us, a
    // head / both: 32 x 56 x 96 x 128, S = 8, k = 2 (168 keys) 143 / 133 with a given index, 27 x 63 x 70 x 192, k = 1 (90) 171 / 163, 15 x 176 x 128 x 64, S = 16, k = 4 (352)
    // 163 / 156; mean of 232 with up to 192 keys 1.028, of 176 with up to 512 1.010; from 11 blocks of keys on, or few workgroups, the other way: 0.99; 4 x 48 x 112 x 128, S = 8,
    // k = 1 38.1 / 39.2).  One query tile: from four workgroups per compute unit on (30 x 42 x 42 x 192, k = 5 107.5 / 103.9; 1 x 72 x 72 x 192, S = 8, k = 12 44.3 / 47.9, 1 x
    // 100 x 150 x 64, S = 16, k = 8 41.8 / 44.7)
    const int t64 = (D.n + 63) / 64, t128 = (D.n + 127) / 128;
    const long regions = (long)D.B * D.R * (D.C / 64), wide = regions * t128;
    if (t128 * 128 * 8 <= t64 * 64 * 9 && wide >= 512) {
        if (D.kn <= 512 && wide >= (D.kn <= 192 ? 768 : 2048)) launch_attn_gen_t<2, 2>(D, A, O, Low, out, st);
        else launch_attn_gen_t<2, 1>(D, A, O, Low, out, st);
    } else if (regions * t64 >= 1024) launch_attn_gen_t<1, 2>(D, A, O, Low, out, st);
    else launch_attn_gen_t<1, 1>(D, A, O, Low, out, st);
}

// Pooling, region-level projections, A^r rows and top-k on their own, for regions of more than one token.
int route_pooled(const Dims &D, const bf16_t *X, const bf16_t *Wqkv, const WideWs &w, int32_t *Ir, float *Ar_opt, hipStream_t st)
{
    launch_pool(D, X, w, GemmRows{}, st);
    const int rc = gemm_regions(region_job(D, w), Wqkv, 3 * D.C, D.C, K_MFMA_ROUTE_ROWS, st);
    return rc == BRA_OK ? route_rows(D, w.qr, w.kr, D.C, Ir, Ar_opt, st) : rc;
}

int route_steps(const Dims &D, const bf16_t *X, const bf16_t *Wqkv, const WideWs &w, int32_t *Ir, float *Ar_opt,
                hipStream_t st)
{
    if (means_from_projection(D)) {               // Q and K themselves are not stored
        const int rc = gemm_means(X, Wqkv, 3 * D.C, D.C, 2 * D.C, GemmOut{{nullptr, nullptr, nullptr}, D.C, {nullptr, nullptr}, nullptr, nullptr, 0},
                                  means_job(D, w, 0, 0), K_MFMA_ROUTE_ROWS, st);
        return rc == BRA_OK ? route_rows(D, w.qr, w.kr, D.C, Ir, Ar_opt, st) : rc;
    }
    if (D.n > 1) return route_pooled(D, X, Wqkv, w, Ir, Ar_opt, st);
    // one token per region: the means are the (bf16) tokens themselves, so Q^r | K^r is the plain projection of X
    // with float32 results: no pooling, no split.  The same product as in wide_forward (a sum's order does not
    // depend on the tile), so that both decide on the same bits
    const int rc = gemm(X, Wqkv, 3 * D.C, (long)D.B * D.R, D.C, 2 * D.C, GemmOut{{w.q, w.k, nullptr}, D.C, {w.qr, w.kr}, nullptr, nullptr, 0}, nullptr,
                        K_MFMA_ROUTE_ROWS, st);
    return rc == BRA_OK ? route_rows(D, w.qr, w.kr, D.C, Ir, Ar_opt, st) : rc;
}

}  // namespace

bool wide_supported(const Dims &D)
{
    if (D.dtype != BRA_BF16 || D.C % 64 != 0 || D.C > 4096) return false;
    if (D.d != 32 && D.d != 64) return false;
    if (many_regions(D) && !generic_supported(D)) return false;               // top-k by the generic kernel
    if (((long)D.B * D.N + 63) / 64 * ((3L * D.C + 127) / 128) > 0x7fffffffL) return false;
    if ((long)D.B * D.R * ((D.n + 63) / 64) * (D.C / 64) > 0x7fffffffL) return false;
    return true;
}

// LCE(V) in front, to which the attention adds itself: what the convolution needs is there as soon as the
// routing's input is, and the routing leaves most of the chip idle.  It is kept in float32: rounded to bf16 it put 7 to 9 %
// on the layer's error from float64, now 3 to 4 % below that of the convolution added to a rounded attention.  On large maps its
// 4 bytes more per value cost more than that hides: beyond 9 million values, or 6 where the rows of the routing are short.  Between the
// two 256 regions gain, 64 regions break even or lose up to 4 % and keep the better precision.  Layer, behind / in front (us), by millions
// of values: 1 x 32 x 32 x 768, k = 12 52.2 / 47.4, 8 of them: 6 115 / 109, 10: 7.5 140 / 136; S = 16: 2 x 200 x 300 x 64 7.3 120 / 117, 1 x
// 250 x 180 x 128 5.5 98 / 91; 20 x 28 x 28 x 512 7.7 107 / 106; 48 x 14 x 14 x 768 6.9 148.5 / 150; 24 x 28 x 28 x 384 6.9 89.5 / 90.6; 20 x 40
// x 40 x 256, S = 8 7.8 92 / 96.  Short rows: 64 x 42 x 42 x 64, k = 4 6.9 76.3 / 78.6; 64 x 21 x 21 x 256 6.9 97 / 100; 48 x 28 x 28 x 192
// 6.9 76.8 / 81.9; 28 x 49 x 49 x 64 4.1 59.4 / 57.7.  Beyond: 64 x 21 x 21 x 384 10.3 148 / 163; 16 x 64 x 64 x 384 24 244 / 274.
// At any size where other kernels take the shape that round O once: with the convolution behind, O is rounded twice, 3.3e-3
// from float64 for 2.87e-3 where the convolution is a third of the attention (5 x 128 x 128 x 128, S = 16, k = 1, equal scores).
bool convolution_in_front(const Dims &D)
{
    return (long)D.B * D.N * D.C <= (D.R * D.C >= 14 << 10 ? 9L : 6L) << 20 || layer_rounds_once(D);
}

size_t wide_workspace_bytes(const Dims &D) { return carve(D, nullptr).bytes; }

int wide_route(const Dims &D, const void *X, const void *Wqkv, int32_t *Ir, float *Ar_opt, void *ws,
               hipStream_t st)
{
    const WideWs w = carve(D, ws);
    return route_steps(D, (const bf16_t *)X, (const bf16_t *)Wqkv, w, Ir, Ar_opt, st);
}

size_t wide_means_bytes(const Dims &D) { return 3 * align256((size_t)D.B * D.R * D.C * 4); }

// The index of wide_route and wide_forward, bit for bit, in less scratch (regions of more than one token).
int wide_route_far(const Dims &D, const void *X, const void *Wqkv, int32_t *Ir, float *Ar_opt, void *means, hipStream_t st)
{
    const size_t each = wide_means_bytes(D) / 3;
    WideWs w = {};
    w.xr = (float *)means;
    w.qr = (float *)((char *)means + each);
    w.kr = (float *)((char *)means + 2 * each);
    return route_steps(D, (const bf16_t *)X, (const bf16_t *)Wqkv, w, Ir, Ar_opt, st);
}

// H, W: the caller's map where D describes a zero-padded one (0: it does not): the products and the pooling read tokens
// beyond it as zeros and do not write them; nothing is copied.  Yp: scratch of the padded map's size then.
int wide_forward(const Dims &D, const void *X, const void *Wqkv, const void *Wo, const void *Wlce, void *Y,
                 int32_t *Ir_out_opt, const int32_t *Ir_in_opt, void *ws, hipStream_t st, int H, int W, void *Yp)
{
    const GemmRows pad = H ? GemmRows{D.H, D.W, H, W} : GemmRows{};
    const WideWs w = carve(D, ws);
    bf16_t *low = (bf16_t *)(H ? Yp : Y);        // nothing else is there until the last product, and X has been read by then
    const int32_t *Ir_src = Ir_in_opt;
    int32_t *Ir_dst = Ir_out_opt ? Ir_out_opt : w.ir;
    // Q^r | K^r: one token per region: Q, K before their rounding to bf16, which the token projection leaves as float32
    // copies; else the projection of the region means, in the same launch as the tokens' (on its own it was a chain of
    // 12 chunks on a few workgroups: 13.7 us at C = 768)
    const long M = (long)D.B * D.N;
    const bool route = !Ir_in_opt, means = route && means_from_projection(D), pooled = route && !means && D.n > 1;
    if (pooled) launch_pool(D, (const bf16_t *)X, w, pad, st);
    const GemmRegions rj = region_job(D, w);
    const float c_exp = D.scale * 1.4426950408889634f;
    const float q_scale = map_tail_pays(D) ? 1.0f : c_exp;     // k_attn_rows, k_attn_gen take scores in units of log2
    const bool copies = route && D.n == 1;
    const GemmOut qkv = {{w.q, w.k, w.v}, D.C, {copies ? w.qr : nullptr, copies ? w.kr : nullptr}, nullptr, nullptr, 0, q_scale, pad, GemmRows{}};
    int rc = means ? gemm_means((const bf16_t *)X, (const bf16_t *)Wqkv, 3 * D.C, D.C, 3 * D.C, qkv, means_job(D, w, H, W), K_MFMA_QKV, st)
                   : gemm((const bf16_t *)X, (const bf16_t *)Wqkv, 3 * D.C, M, D.C, 3 * D.C, qkv, pooled ? &rj : nullptr, K_MFMA_QKV, st);
    if (rc != BRA_OK) return rc;
    AttnArgs A = {};
    bool adds = false;
    const bool map_tail = map_tail_pays(D);      // forms the LCE itself
    if (!map_tail && convolution_in_front(D)) {
        rc = lce::route_rows_lce_bf16(D, route ? w.qr : nullptr, w.kr, Ir_dst, w.v, (const bf16_t *)Wlce, w.o, low, st);
        if (rc != BRA_OK && rc != BRA_ERR_UNSUPPORTED) return rc;
        adds = rc == BRA_OK;
    }
    if (route && !adds) {
        rc = route_rows(D, w.qr, w.kr, D.C, Ir_dst, nullptr, st);
        if (rc != BRA_OK) return rc;
    }
    if (route) Ir_src = Ir_dst;
    A.X = (const bf16_t *)X; A.Q = w.q; A.K = w.k; A.V = w.v;
    A.Ir_src = Ir_src; A.Ir_out = Ir_out_opt; A.Wlce = (const bf16_t *)Wlce; A.Y = (bf16_t *)Y;
    A.c_exp = c_exp;
    if (map_tail) {
        rc = launch_map_tail(D, A, w.o, st);
    } else {
        {
            ProfScope ps(st, K_MFMA_ATTENTION);
            if (D.n <= 32 && D.k <= 1024) rc = launch_attn_rows(D, A, w.o, adds ? low : nullptr, st);      // its tables fit in LDS
            else {
                const bool with_out = adds && D.C == 64 && D.d == 32;
                launch_attn_gen(D, A, w.o, adds ? low : nullptr, with_out ? OutMap{(const bf16_t *)Wo, (bf16_t *)Y, H, W} : OutMap{}, st);
                if (with_out) return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
            }
        }
        if (rc != BRA_OK) return rc;
        rc = adds ? BRA_OK : lce::lce_add_bf16(D, w.v, (const bf16_t *)Wlce, w.o, D.C, K_MFMA_LCE_ADD, st);
    }
    if (rc != BRA_OK) return rc;
    return gemm(w.o, (const bf16_t *)Wo, D.C, M, D.C, D.C,
                GemmOut{{Y, nullptr, nullptr}, D.C, {nullptr, nullptr}, nullptr, nullptr, 0, 1.0f, GemmRows{}, pad}, nullptr, K_MFMA_WO, st);
}

}  // namespace bra
