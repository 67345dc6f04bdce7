// Region-level routing from float32 Q^r, K^r (Sec. 3.2): rows of A^r = Q^r (K^r)^T (Eq. 4) on the float32
// matrix-core instruction and their top-k (Eq. 5), for any channel count and up to 1024 regions.
//
// Workgroup = (image, 16 query regions), 8 wavefronts.  A pass covers 64 KGP key regions: wavefront w takes key
// group w / CS (4 tiles of 16 regions) and every CS-th step of 16 channels, with all operands straight from memory
// (16 bytes per lane and row; the tensors sit in the L2 of the launch before); the channel slices meet in LDS and
// are added in a fixed order.  Then each wavefront ranks 2 of the rows.
// The work is tiny (50 MFLOP for 8 x 64 regions of 768 channels) and was bound by a chain of 12 staged channel
// chunks, about a microsecond each (13.5 us); here the chain is one round of loads, one reduction, one ranking.
#pragma once

#include "bra_mfma_dev.h"

#include <algorithm>
#include <type_traits>

namespace bra {
namespace route {

using mfma::f32x4;
using mfma::kWave;
using mfma::topk_order_key;
using mfma::wave_topk_rows;
using mfma::wave_umax;

constexpr int kRows = 16, kWaves = 8, kPitch = 64 + 4;
constexpr int kMaxSlots = 16;       // entries of a row per lane: R <= 64 * 16

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float *p, int left)
{
    if (VEC) return *(const f32x4 *)p;
    return f32x4{left > 0 ? p[0] : 0.f, left > 1 ? p[1] : 0.f, left > 2 ? p[2] : 0.f, left > 3 ? p[3] : 0.f};
}

// The k largest of a row of R > 64 entries, lane j holding entries j, j + 64, ..: rounds of wavefront maximum over
// the entries not taken yet, the lowest index among equal values (order as in wave_topk).
template <int SLOTS>
__device__ __forceinline__ void topk_wide(const float *row, int R, int k, int lane, int32_t *out)
{
    uint32_t key[SLOTS];
#pragma unroll
    for (int t = 0; t < SLOTS; ++t) {
        const int j = lane + 64 * t;
        key[t] = j < R ? topk_order_key(row[j], j, R) : 0u;         // a value's key is never 0
    }
    for (int p = 0; p < k; ++p) {
        uint32_t best = 0u;
        int at = 0;
#pragma unroll
        for (int t = 0; t < SLOTS; ++t)
            if (key[t] > best) { best = key[t]; at = t; }
        const uint32_t m = wave_umax(best);
        // lowest index among the holders: the largest complement
        const int j = lane + 64 * at;
        const int first = 0x7fffffff - (int)wave_umax(best == m ? (uint32_t)(0x7fffffff - j) : 0u);
        if (lane == 0) out[p] = first;
#pragma unroll
        for (int t = 0; t < SLOTS; ++t)
            if (first == lane + 64 * t) key[t] = 0u;
    }
}

// VEC: C and ld multiples of 4 (16-byte loads).  PART: C may not be a multiple of 16.  CS, KGP: channel slices and key
// groups per pass, CS * KGP = 8.  Called by 64 kWaves threads.
// MOST: steps requested at once.  The sums do not depend on it, infinities and NaN included: bra_route and bra_forward take
// different ones, and a step repeated past the end with blanked queries alone made NaN of an infinite K^r in one and not the other.
// As many steps as are left, no more (bra_route of 2 x 14 x 14 x 512, four steps: 23.5 us with six, 21.8); beside the convolution
// one by one after the threes (code for two as well: 2 x 8 x 24 x 512 33.9 us, 33.5 without; 11 x 7 x 7 x 768 39.4 and 38.9).
template <bool VEC, bool PART, int MOST>
__device__ __forceinline__ void route_block(const float *__restrict__ Qr, const float *__restrict__ Kr, int ld, int32_t *__restrict__ Ir,
                                            float *__restrict__ Ar, const Dims &D, int CS, int block, float *smem)
{
    float *red = smem;                                  // [wavefront][16 rows][kPitch]
    float *rows = smem + kWaves * kRows * kPitch;       // [16][row pitch]: the rows of A^r
    const int KGP = kWaves / CS, groups = (D.R + 63) / 64, pitch = 64 * groups + 4;
    const int rtiles = (D.R + kRows - 1) / kRows, b = block / rtiles, r0 = (block % rtiles) * kRows;
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int cs = w % CS, steps = (D.C + 15) / 16;
    const size_t img = (size_t)b * D.R * ld;
    const float *qrow = Qr + img + (size_t)min(r0 + i, D.R - 1) * ld;
    for (int kg0 = 0; kg0 < groups; kg0 += KGP) {
        const int kg = kg0 + w / CS;
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (kg < groups) {
            const float *krow[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) krow[t] = Kr + img + (size_t)min(64 * kg + 16 * t + i, D.R - 1) * ld;
            // NB steps at once: their loads are all requested before the first product
            auto batch = [&](int s, auto nb) {
                constexpr int NB = decltype(nb)::value;
                f32x4 q[NB], kv[NB][4];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int c = 16 * min(s + u * CS, steps - 1) + 4 * g, cc = VEC ? min(c, D.C - 4) : c;
                    q[u] = load4<VEC>(qrow + cc, D.C - c);
#pragma unroll
                    for (int t = 0; t < 4; ++t) kv[u][t] = load4<VEC>(krow[t] + cc, D.C - c);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    // channels past the end, in the last of all steps alone: blanked on both sides
                    const bool past = 16 * (s + u * CS) + 4 * g >= D.C;
                    if (past) q[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (VEC && PART && u == NB - 1) {
#pragma unroll
                        for (int t = 0; t < 4; ++t) kv[u][t] = past ? f32x4{0.f, 0.f, 0.f, 0.f} : kv[u][t];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[t] = mfma_f32(q[u][e], kv[u][t][e], acc[t]);   // D[query 4 g + j][key i]
                }
            };
            for (int s = cs; s < steps;) {
                const int left = (steps - s + CS - 1) / CS;
                auto take = [&](auto nb) {
                    batch(s, nb);
                    s += decltype(nb)::value * CS;
                };
                if (left >= MOST) take(std::integral_constant<int, MOST>{});
                else if (MOST > 5 && left == 5) take(std::integral_constant<int, 5>{});
                else if (MOST > 4 && left == 4) take(std::integral_constant<int, 4>{});
                else if (MOST > 3 && left == 3) take(std::integral_constant<int, 3>{});
                else if (MOST > 3 && left == 2) take(std::integral_constant<int, 2>{});
                else take(std::integral_constant<int, 1>{});
            }
        }
        if (kg0) __syncthreads();                        // the previous pass has been added up
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[(w * kRows + 4 * g + j) * kPitch + 16 * t + i] = acc[t][j];
        __syncthreads();
        for (int e = tid; e < KGP * kRows * 64; e += 64 * kWaves) {
            const int col = e % 64, row = (e / 64) % kRows, kq = e / (64 * kRows);
            float s = 0.f;
            for (int u = 0; u < CS; ++u) s += red[((kq * CS + u) * kRows + row) * kPitch + col];
            if (kg0 + kq < groups) rows[row * pitch + 64 * (kg0 + kq) + col] = s;
        }
    }
    __syncthreads();
    const size_t out0 = (size_t)b * D.R + r0;
    if (Ar) {
        for (int row = w; row < kRows && r0 + row < D.R; row += kWaves)
            for (int j = lane; j < D.R; j += 64) Ar[(out0 + row) * D.R + j] = rows[row * pitch + j];
    }
    const int first = 2 * w, nrows = min(2, D.R - r0 - first);
    if (nrows <= 0) return;
    if (groups == 1) {
        const float v[2] = {rows[first * pitch + lane], rows[(first + 1) * pitch + lane]};
        wave_topk_rows<2>(v, nrows, lane, D.R, D.k, Ir + (out0 + first) * D.k);
    } else {
        for (int rr = 0; rr < nrows; ++rr) {
            const float *row = rows + (first + rr) * pitch;
            int32_t *out = Ir + (out0 + first + rr) * D.k;
            if (groups <= 4) topk_wide<4>(row, D.R, D.k, lane, out);
            else topk_wide<kMaxSlots>(row, D.R, D.k, lane, out);
        }
    }
}


struct Plan {
    int CS, blocks;
    size_t smem;
    bool vec;
};

inline Plan plan(const Dims &D, int ld)
{
    const int steps = (D.C + 15) / 16, groups = (D.R + 63) / 64;
    // channel slices: as many as there are steps, but no more than leaves work for all wavefronts on the key groups
    Plan p;
    p.CS = kWaves;
    while (p.CS > 1 && (p.CS > steps || kWaves / p.CS < std::min(groups, 4))) p.CS /= 2;
    p.smem = (size_t)(kWaves * kRows * kPitch + kRows * (64 * groups + 4)) * sizeof(float);
    p.vec = D.C % 4 == 0 && ld % 4 == 0;
    p.blocks = (int)((long)D.B * ((D.R + kRows - 1) / kRows));
    return p;
}

inline bool supported(const Dims &D) { return D.R <= kWave * kMaxSlots; }

}  // namespace route
}  // namespace bra
