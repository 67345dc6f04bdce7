// Attention gradients in float32 for regions of at most 32 tokens and heads of at most 32 channels: W wavefronts share a head of a
// region, each with every Wth tile of 16 rows of the other side, and add up through LDS at the end.  (internal)
//
// A wavefront brings its rows by itself, once as the operand whose rows they are and through its own part of LDS as the one whose columns
// they are; there is no barrier but for the sums.  What bounded the kernels that stage 32 or 64 rows of four heads for the
// whole workgroup: one wavefront per head with a chain of loads, barriers and products per block, and on the key side the most
// popular region's list on one compute unit.  Whole gradient, us, with those and so: 8 x 28 x 28 x 128, k = 4 82.9 -> 74.4 (query side with the tap
// gradients' pass 20.6 -> 18.1, key side 25.2 -> 16.8); 3 x 32 x 32 x 128, S = 16, k = 11 80.9 -> 73.6; 12 x 24 x 24 x 64, S = 8, k = 30 160 -> 95; bf16 4 x 14 x 28 x
// 96, k = 16 66.9 -> 43.8; 60 x 28 x 28 x 96, k = 4 270 -> 252; 16 x 35 x 35 x 96, k = 8 304 -> 257.  A pass with two channels per thread would take 190
// registers and leave two wavefronts per SIMD.
#pragma once

#include "bra_f32_dev.h"

#include <cfloat>

namespace bra {
namespace f32 {

template <int W>
struct HeadShare {
    static constexpr int P = 32 + 4, HPG = 4 / W, kTile = 16 * P;      // heads of a workgroup; floats of a tile of rows in LDS
};

// Between what lanes of a wavefront write to its part of LDS and what others of it read there, both ways.  No instruction: the hardware keeps
// the order of a wavefront's accesses, this asks the compiler to.
__device__ __forceinline__ void lanes_meet() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Sums over the W wavefronts of a head: v of wavefront `part` goes to sums[..][part]; behind a barrier, total() adds them up in order.
// N f32x4 per lane; entry c of all wavefronts is taken by wavefront c % W.
template <int W, int N>
__device__ __forceinline__ void park_parts(f32x4 *sums, int hl, int part, int lane, const f32x4 (&v)[N])
{
#pragma unroll
    for (int c = 0; c < N; ++c) sums[((hl * N + c) * W + part) * 64 + lane] = v[c];
}
template <int W, int N>
__device__ __forceinline__ f32x4 total(const f32x4 *sums, int hl, int lane, int c, const float *f = nullptr)
{
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const f32x4 x = sums[((hl * N + c) * W + w) * 64 + lane];
        t += f ? x * f[w] : x;
    }
    return t;
}

// Query side, see k_attn_bwd_q: O, lse, D and dQ of NQ tiles of 16 queries.  The weights and dP of up to kKept tiles of keys per
// wavefront stay in registers; of more, they are formed twice.  Scores are scaled behind their products, here and on the key side, and rounded once: the
// statistics belong to the very scores that the key side forms, and terms that cancel do.
// Four wavefronts per SIMD, which spill 2 and 4 registers where two wavefronts or one have a head; three, which spill none: 8 x 28 x 28 x 128, k = 4 74.3 -> 73.9 us, 6 images 69.3 -> 70.2, 12 images
// 102.9 -> 103.4.
template <int NQ>
constexpr int kKeptTiles = NQ == 1 ? 4 : 2;

template <int NQ, int W, bool VEC>
__global__ __launch_bounds__(256, NQ == 1 && VEC ? 4 : 3) void k_heads_bwd_q(const float *__restrict__ QKV, const float *__restrict__ dO, const int32_t *__restrict__ Ir,
                                                     float *__restrict__ O, float *__restrict__ dQKV, float *__restrict__ lse, float *__restrict__ dsum,
                                                     Dims D, int hgroups, bool by_image, lce::GradJob<float> J, int lce_blocks)
{
    typedef HeadShare<W> L;
    constexpr int kKept = kKeptTiles<NQ>;
    constexpr int P = L::P, NS = 2, kRows = 4 * 2 * L::kTile, kSums = W > 1 ? 4 * NQ * NS * 64 * 4 : 0, kFloats = kRows + kSums > 25 * 256 ? kRows + kSums : 25 * 256;
    __shared__ __attribute__((aligned(16))) float lds[kFloats];
    __shared__ float stats[W > 1 ? 4 * NQ * 3 * 16 : 1];
    int wg, wgs;
    if (lce::block_of_pass(lce_blocks, false, wg, wgs)) {
        lce::lce_grad_block<1, false>(J, D, mfma::swizzled(wg, wgs), lds);
        return;
    }
    const AttnWork work = attn_work(wg, wgs, by_image, 1, hgroups, D.R);
    const int reg = work.region, b = work.image;
    if (b >= D.B) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave, g = lane / 16, i = lane % 16;
    const int hl = wave / W, part = wave % W, h = work.hg * L::HPG + hl, C3 = 3 * D.C, kn = D.kn, tiles = (kn + 15) / 16;
    const bool head = h < D.heads;
    const size_t itok = (size_t)b * D.N;
    const float *img = QKV + itok * C3;
    const int32_t *irp = Ir + ((size_t)b * D.R + reg) * D.k;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n, c_exp = D.scale * 1.4426950408889634f;
    float *Kw = lds + wave * 2 * L::kTile, *Vw = Kw + L::kTile;
    f32x4 *sums = (f32x4 *)(lds + kRows);
    auto row_chunk = [&](const float *row, int s) { return load_head_chunk<32, VEC>(row, 4 * s + g, h, D); };
    auto blank = [&](f32x4 v, int s) { return blank_head_chunk<32, VEC>(v, 4 * s + g, h, D); };
    int qtok[NQ];
    f32x4 qf[NQ][NS], gf[NQ][NS];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        qtok[q] = at.origin(reg) + at.slot(min(16 * q + i, D.n - 1));
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            qf[q][s] = blank(row_chunk(img + (size_t)qtok[q] * C3, s), s);
            gf[q][s] = blank(row_chunk(dO + (itok + qtok[q]) * D.C, s), s);
        }
    }
    f32x4 kr[NS], vr[NS];
    auto fetch = [&](int tile, bool both) {
        const int key = min(16 * tile + i, kn - 1), p = divide(key, D.n, n_inv);      // past the end: the last key, masked below
        const float *row = img + (size_t)(at.origin(region_index(irp[p], D.R)) + at.slot(key - p * D.n)) * C3;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            kr[s] = row_chunk(row + D.C, s);
            if (both) vr[s] = row_chunk(row + 2 * D.C, s);
        }
    };
    auto park_keys = [&](f32x4 (&k)[NS]) {
        lanes_meet();                            // the tile before has been read
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            k[s] = blank(kr[s], s);
            *(f32x4 *)(Kw + i * P + 16 * s + 4 * g) = k[s];
        }
    };
    // The scores and dP of a tile of keys; K, and V with `both`, go to LDS.
    f32x4 st[kKept][NQ], dp[kKept][NQ];
    auto scores = [&](int tile, bool both, f32x4 (&st)[NQ], f32x4 (&dp)[NQ]) {
        f32x4 k[NS], v[NS];
        park_keys(k);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            v[s] = blank(vr[s], s);
            if (both) *(f32x4 *)(Vw + i * P + 16 * s + 4 * g) = v[s];
        }
        lanes_meet();
        if (tile + W < tiles) fetch(tile + W, true);
#pragma unroll
        for (int q = 0; q < NQ; ++q) st[q] = dp[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    st[q] = mfma_f32(k[s][e], qf[q][s][e], st[q]);          // S^T[key 4 g + j][query i]
                    dp[q] = mfma_f32(v[s][e], gf[q][s][e], dp[q]);
                }
        const int left = kn - 16 * tile;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[q][j] = 4 * g + j < left ? st[q][j] : -INFINITY;
    };
    f32x4 acc[NQ * NS];
    auto contract = [&](const float *T, const f32x4 (&wt)[NQ]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < NS; ++dt) {
                const float t = T[(4 * g + e) * P + 16 * dt + i];
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[NS * q + dt] = mfma_f32(t, wt[q][e], acc[NS * q + dt]);
            }
    };
    float m[NQ], l[NQ], dd[NQ];                 // m: an exponent of 2, at first a finite one: a tile without a finite score leaves no weights, and no NaN
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        m[q] = -FLT_MAX;
        l[q] = dd[q] = 0.f;
#pragma unroll
        for (int dt = 0; dt < NS; ++dt) acc[NS * q + dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float then[kKept][NQ];                       // the reference that a kept tile's weights have
    if (part < tiles) fetch(part, true);
    for (int t0 = part; t0 < tiles; t0 += kKept * W) {
#pragma unroll
        for (int u = 0; u < kKept; ++u) {
            if (t0 + u * W >= tiles) break;
            scores(t0 + u * W, true, st[u], dp[u]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                f32x4 &x = st[u][q];
                const float top = fmaxf(m[q], cross_row_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]))) * c_exp);
                const float alpha = __builtin_amdgcn_exp2f(m[q] - top);
                m[q] = then[u][q] = top;
                float ls = 0.f, ds = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[j] = __builtin_amdgcn_exp2f(fmaf(x[j], c_exp, -top));
                    ls += x[j];
                    ds = fmaf(x[j], dp[u][q][j], ds);
                }
                l[q] = fmaf(l[q], alpha, ls);    // this lane's keys; the lane groups meet below
                dd[q] = fmaf(dd[q], alpha, ds);
#pragma unroll
                for (int dt = 0; dt < NS; ++dt) acc[NS * q + dt] *= alpha;
            }
            contract(Vw, st[u]);
        }
    }
    const bool twice = tiles > kKept * W;
    if (part < tiles) fetch(part, twice);
    // all wavefronts' sums on a common reference
    float inv[NQ], fs[NQ][W];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        l[q] = cross_row_sum(l[q]);
        dd[q] = cross_row_sum(dd[q]);
    }
    if constexpr (W > 1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (g == 0) {
                float *to = stats + ((hl * W + part) * NQ + q) * 48 + i;
                to[0] = m[q];
                to[16] = l[q];
                to[32] = dd[q];
            }
        park_parts<W, NQ * NS>(sums, hl, part, lane, acc);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            float top = -FLT_MAX;
            const float *from = stats + (hl * W * NQ + q) * 48 + i;
#pragma unroll
            for (int w = 0; w < W; ++w) top = fmaxf(top, from[w * NQ * 48]);
            l[q] = dd[q] = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                fs[q][w] = __builtin_amdgcn_exp2f(from[w * NQ * 48] - top);
                l[q] = fmaf(from[w * NQ * 48 + 16], fs[q][w], l[q]);
                dd[q] = fmaf(from[w * NQ * 48 + 32], fs[q][w], dd[q]);
            }
            m[q] = top;
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        inv[q] = 1.0f / l[q];
        dd[q] *= inv[q];
        if (head && part == 0 && g == 0 && 16 * q + i < D.n) {
            lse[(itok + qtok[q]) * D.heads + h] = m[q] + __builtin_amdgcn_logf(l[q]);    // v_log_f32: log2
            dsum[(itok + qtok[q]) * D.heads + h] = dd[q];
        }
    }
    auto store = [&](float *rows, size_t ld, const float (&scale)[NQ], bool weighted) {
#pragma unroll
        for (int c = 0; c < NQ * NS; ++c) {
            if (c % W != part) continue;
            const int q = c / NS, dt = c % NS, ch = 16 * dt + 4 * g;
            const f32x4 v = W > 1 ? total<W, NQ * NS>(sums, hl, lane, c, weighted ? fs[q] : nullptr) : acc[c];
            if (head && 16 * q + i < D.n && ch < D.d) store4<VEC>(rows + qtok[q] * ld + h * D.d + ch, v * scale[q], D.d - ch);
        }
    };
    store(O + itok * D.C, D.C, inv, true);
#pragma unroll
    for (int c = 0; c < NQ * NS; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t0 = part; t0 < tiles; t0 += kKept * W) {
#pragma unroll
        for (int u = 0; u < kKept; ++u) {
            const int tile = t0 + u * W;
            if (tile >= tiles) break;
            if (twice) {
                scores(tile, false, st[u], dp[u]);
            } else {
                f32x4 k[NS];
                park_keys(k);
                lanes_meet();
                if (tile + W < tiles) fetch(tile + W, false);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const float f = twice ? 1.0f : __builtin_amdgcn_exp2f(then[u][q] - m[q]);
#pragma unroll
                for (int j = 0; j < 4; ++j) st[u][q][j] = (twice ? __builtin_amdgcn_exp2f(fmaf(st[u][q][j], c_exp, -m[q])) : st[u][q][j] * f) * inv[q] * (dp[u][q][j] - dd[q]);
            }
            contract(Kw, st[u]);
        }
    }
    if constexpr (W > 1) {
        __syncthreads();                         // the sums have been read
        park_parts<W, NQ * NS>(sums, hl, part, lane, acc);
        __syncthreads();
    }
    float scale[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) scale[q] = D.scale;
    store(dQKV + itok * C3, C3, scale, false);
}

// Key side, see k_attn_bwd_kv: dK and dV of NK tiles of 16 keys, over the rows of all query regions routed to the region.
template <int NK, int W, bool VEC>
__global__ __launch_bounds__(256, NK == 1 ? 4 : 3) void k_heads_bwd_kv(const float *__restrict__ QKV, const float *__restrict__ dO, const int32_t *__restrict__ Ir,
                                                      const float *__restrict__ lse, const float *__restrict__ dsum, float *__restrict__ dQKV, Dims D,
                                                      int hgroups, bool by_image, lce::AddJob<float> J, int lce_blocks)
{
    typedef HeadShare<W> L;
    constexpr int P = L::P, NS = 2, kWaveFloats = 2 * L::kTile + 32, kRows = 4 * kWaveFloats, kSums = W > 1 ? 4 * NK * 2 * NS * 64 * 4 : 0;
    __shared__ __attribute__((aligned(16))) float lds[kRows > kSums ? kRows : kSums];        // the rows, then the sums
    __shared__ int list[bwd::kListChunk], counts[16];
    static_assert(kRows >= 25 * 64, "the pass shares the buffers");
    int wg, wgs;
    if (lce::block_of_pass(lce_blocks, false, wg, wgs)) {
        lce::lce_block<VEC ? 2 : 1, true, 256>(J, D, mfma::swizzled(wg, wgs), lds);
        return;
    }
    const AttnWork work = attn_work(wg, wgs, by_image, 1, hgroups, D.R);
    const int reg = work.region, b = work.image;
    if (b >= D.B) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave, g = lane / 16, i = lane % 16;
    const int hl = wave / W, part = wave % W, h = work.hg * L::HPG + hl, C3 = 3 * D.C;
    const bool head = h < D.heads;
    const size_t itok = (size_t)b * D.N;
    const float *img = QKV + itok * C3;
    const Places<true> at(D);
    const float n_inv = 1.0f / (float)D.n, k_inv = 1.0f / (float)D.k, c_exp = D.scale * 1.4426950408889634f;
    float *Qw = lds + wave * kWaveFloats, *Gw = Qw + L::kTile, *lw = Gw + L::kTile;
    auto row_chunk = [&](const float *row, int s) { return load_head_chunk<32, VEC>(row, 4 * s + g, h, D); };
    auto blank = [&](f32x4 v, int s) { return blank_head_chunk<32, VEC>(v, 4 * s + g, h, D); };
    int ktok[NK];
    f32x4 kf[NK][NS], vf[NK][NS], sum[2 * NK * NS];      // [tile][dK, dV][channels]
#pragma unroll
    for (int q = 0; q < NK; ++q) {
        ktok[q] = at.origin(reg) + at.slot(min(16 * q + i, D.n - 1));
        const float *row = img + (size_t)ktok[q] * C3;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            kf[q][s] = blank(row_chunk(row + D.C, s), s);
            vf[q][s] = blank(row_chunk(row + 2 * D.C, s), s);
        }
    }
#pragma unroll
    for (int c = 0; c < 2 * NK * NS; ++c) sum[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int entries = D.R * D.k;
    const int32_t *irb = Ir + (size_t)b * entries;
    f32x4 qr[NS], gr[NS];
    float row_lse, row_dd;                       // of row i of the tile
    for (int e0 = 0; e0 < entries; e0 += bwd::kListChunk) {
        const int rows = bwd::collect_entries(irb, entries, e0, reg, D.R, list, counts) * D.n;
        auto fetch = [&](int tile) {
            const int row = min(16 * tile + i, rows - 1), e = divide(row, D.n, n_inv);
            const int tok = at.origin(divide(list[e], D.k, k_inv)) + at.slot(row - e * D.n);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                qr[s] = row_chunk(img + (size_t)tok * C3, s);
                gr[s] = row_chunk(dO + (itok + tok) * D.C, s);
            }
            const size_t st = (itok + tok) * D.heads + (head ? h : 0);
            row_lse = lse[st];
            row_dd = dsum[st];
        };
        if (16 * part < rows) fetch(part);
        for (int tile = part; 16 * tile < rows; tile += W) {
            f32x4 qv[NS], gv[NS];
            lanes_meet();                        // the tile before has been read
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                qv[s] = blank(qr[s], s);
                gv[s] = blank(gr[s], s);
                *(f32x4 *)(Qw + i * P + 16 * s + 4 * g) = qv[s];
                *(f32x4 *)(Gw + i * P + 16 * s + 4 * g) = gv[s];
            }
            if (g == 0) {
                lw[i] = 16 * tile + i < rows ? row_lse : INFINITY;       // a missing row: P = exp2(-inf) = 0
                lw[16 + i] = row_dd;
            }
            lanes_meet();
            if (16 * (tile + W) < rows) fetch(tile + W);
            f32x4 st[NK], dp[NK];
#pragma unroll
            for (int q = 0; q < NK; ++q) st[q] = dp[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int q = 0; q < NK; ++q) {
                        st[q] = mfma_f32(qv[s][e], kf[q][s][e], st[q]);      // S[query 4 g + j][key i]
                        dp[q] = mfma_f32(gv[s][e], vf[q][s][e], dp[q]);
                    }
            const f32x4 l4 = *(const f32x4 *)(lw + 4 * g), d4 = *(const f32x4 *)(lw + 16 + 4 * g);
            f32x4 p[NK], ds[NK];
#pragma unroll
            for (int q = 0; q < NK; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    p[q][e] = __builtin_amdgcn_exp2f(fmaf(st[q][e], c_exp, -l4[e]));
                    ds[q][e] = p[q][e] * (dp[q][e] - d4[e]);
                }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int dt = 0; dt < NS; ++dt) {
                    const float qc = Qw[(4 * g + e) * P + 16 * dt + i], gc = Gw[(4 * g + e) * P + 16 * dt + i];
#pragma unroll
                    for (int q = 0; q < NK; ++q) {
                        sum[(2 * q) * NS + dt] = mfma_f32(qc, ds[q][e], sum[(2 * q) * NS + dt]);             // dK^T[channel 16 dt + 4 g + j][key i]
                        sum[(2 * q + 1) * NS + dt] = mfma_f32(gc, p[q][e], sum[(2 * q + 1) * NS + dt]);      // dV^T
                    }
                }
        }
    }
    if constexpr (W > 1) {
        __syncthreads();                         // the rows have been read
        park_parts<W, 2 * NK * NS>((f32x4 *)lds, hl, part, lane, sum);
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < 2 * NK * NS; ++c) {
        if (c % W != part) continue;
        const int q = c / (2 * NS), which = c / NS % 2, ch = 16 * (c % NS) + 4 * g;
        const f32x4 v = W > 1 ? total<W, 2 * NK * NS>((const f32x4 *)lds, hl, lane, c) : sum[c];
        if (!head || 16 * q + i >= D.n || ch >= D.d) continue;
        float *to = dQKV + (itok + ktok[q]) * C3 + (1 + which) * D.C + h * D.d + ch;
        store4<VEC>(to, which ? v + load4<VEC>(to, D.d - ch) : v * D.scale, D.d - ch);       // dV: LCE^T(dO) is there
    }
}

}  // namespace f32
}  // namespace bra
