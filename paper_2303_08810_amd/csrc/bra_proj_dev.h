// Tiles of the products with a short contraction, for the kernels that keep all of the weights in LDS (k_proj, k_proj_route).
#pragma once

#include "bra_gemm.h"
#include "bra_mfma_dev.h"

namespace bra {

using mfma::bf16x8;
using mfma::f32x4;
using mfma::kWave;
using mfma::lds_read_tr16;
using mfma::mfma16;
using mfma::pack8;
using mfma::u32x2;
using mfma::u32x4;

// Products with a short contraction (K = 64 or 128) over many rows, into bf16 buffers of K columns each (N = K or 3 K): Q, K,
// V, dO and Y of the first stages.  A tile of k_gemm_dma has one or two chunks to load before it stores, and its loads and
// stores do not overlap with those of the one or two workgroups beside it (150528 x 128 x 384: 52 us, of which 30 without
// the stores and 22 without the loads).  Here a workgroup per compute unit keeps all of W in LDS and its wavefronts walk
// over tiles of 16 rows on their own: a row of In is an operand as it lies (16 bytes per lane, the next tile's on their way),
// and there is no barrier behind the staging of W.
// Two 16-output tiles make 32 outputs of which a lane holds 8 consecutive ones (output 8 i / 4 + 4 half + i % 4 for row i of
// tile `half`).  W's columns lie in LDS in that order, so that a transposing read takes 32 bytes of each of 4 rows; rows are
// 32 bytes longer than their columns and groups of 8 rows 128 bytes apart: the 8 rows of 32 lanes then cover all banks.
// BT: W is given transposed ([N][ldw]) and read as it lies.
template <int K, int N, bool BT>
struct ProjLds {
    static constexpr int pitch = BT ? K + 8 : N + 16;
    static constexpr size_t bytes = BT ? (size_t)N * pitch * 2 : (size_t)(K * pitch + K / 8 * 64) * 2;
};

// W into LDS.
template <int K, int N, bool BT>
__device__ __forceinline__ void proj_stage(bf16_t *Ws, const bf16_t *__restrict__ W, int ldw)
{
    constexpr int P = ProjLds<K, N, BT>::pitch;
    const int T = blockDim.x, tid = threadIdx.x;
    if (BT) {
        for (int e = tid; e < N * (K / 8); e += T) {
            const int o = e / (K / 8), k8 = e % (K / 8);
            *(u32x4 *)(Ws + o * P + 8 * k8) = *(const u32x4 *)(W + (size_t)o * ldw + 8 * k8);
        }
    } else {
        for (int e = tid; e < K * (N / 8); e += T) {
            const int k = e / (N / 8), o8 = e % (N / 8);              // columns 8 q .. 8 q + 7 of a group of 32
            const u32x4 v = *(const u32x4 *)(W + (size_t)k * ldw + 8 * o8);
            bf16_t *dst = Ws + k * P + (k / 8) * 64 + 32 * (o8 / 4) + 4 * (o8 % 4);
            *(u32x2 *)dst = u32x2{v[0], v[1]};
            *(u32x2 *)(dst + 16) = u32x2{v[2], v[3]};
        }
    }
}

// One tile of 16 rows: xf its operands.  again: set anew by the caller for every tile, so that the operands are not kept in
// registers across tiles.
template <int K, int N, bool BT>
__device__ __forceinline__ void proj_tile(const bf16_t *Ws, int again, const bf16x8 (&xf)[K / 32], long t, long M, const GemmOut &out)
{
    constexpr int P = ProjLds<K, N, BT>::pitch, KS = K / 32, TP = N / 32;
    const int lane = threadIdx.x % kWave, g = lane / 16, i = lane % 16;
    auto operand = [&](int tp, int half, int ks) {
        if (BT) return *(const bf16x8 *)(Ws + again + (32 * tp + 8 * (i / 4) + 4 * half + i % 4) * P + 32 * ks + 8 * g);
        const bf16_t *p = Ws + (32 * ks + 8 * g + i / 4) * P + (4 * ks + g) * 64 + 32 * tp + 16 * half + 4 * (i % 4) + again;
        const u32x2 r0 = __builtin_bit_cast(u32x2, lds_read_tr16(p)), r1 = __builtin_bit_cast(u32x2, lds_read_tr16(p + 4 * P));
        return __builtin_bit_cast(bf16x8, u32x4{r0[0], r0[1], r1[0], r1[1]});
    };
    const long m = t * 16 + i;
    const size_t at = (size_t)min(m, M - 1) * K + 8 * g;
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) {
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int half = 0; half < 2; ++half) acc[half] = mfma16(operand(tp, half, ks), xf[ks], acc[half]);
        const float scale = 32 * tp < K ? out.scale0 : 1.0f;
        const float v[8] = {acc[0][0] * scale, acc[0][1] * scale, acc[0][2] * scale, acc[0][3] * scale,
                            acc[1][0] * scale, acc[1][1] * scale, acc[1][2] * scale, acc[1][3] * scale};
        if (m < M) *(bf16x8 *)((bf16_t *)out.buf[32 * tp / K] + at + 32 * tp % K) = pack8(v);
    }
}

}  // namespace bra
