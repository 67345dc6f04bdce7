// Device-side pieces of the routed attention kernels that stream rows straight into LDS (internal).
#pragma once

#include "bra_mfma_dev.h"

#include <type_traits>

namespace bra {
namespace mfma {

// Softmax step for KT tiles of 16 keys x 16 queries of one head: scores
// s[t][j] = S^T[key 16 t + 4 g + j][query i] relative to the reference m (which entered the product as its accumulator
// input, so a score costs no subtraction), weights p = 2^s in the operand order of O^T += V^T P^T.  l: the lane's share of
// the denominator, a sum of the float32 weights (over its keys: the caller adds up the four lane groups at the end).
// That sum also decides when the reference has to move: only when a lane's weights of a block exceed 2^8 together, which
// needs no maximum and no exchange between lanes; the quotient O / l does not depend on it.  FIRST: the reference is this
// block's maximum.  With dp (scores of the gradient in the same layout) also d: the lane's share of sum p dp.
template <bool FIRST, int KT, int NDT>
__device__ __forceinline__ void softmax_step(f32x4 (&s)[KT], float &m, float &l, f32x4 (&acc)[NDT], bf16x8 (&pb)[KT / 2],
                                             const f32x4 *dp = nullptr, float *d = nullptr)
{
    auto raise = [&](bool keep) {               // moves the reference to the largest score; returns by how much
        float mx = s[0][0];
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) mx = fmaxf(mx, s[t][j]);
        const float up = keep ? fmaxf(cross_row_max(mx), 0.f) : cross_row_max(mx);
        m += up;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) s[t][j] -= up;
        return up;
    };
    float dsum = 0.f;
    auto weights = [&]() {
        float sum[2];
        dsum = 0.f;
#pragma unroll
        for (int tp = 0; tp < KT / 2; ++tp) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p[e] = __builtin_amdgcn_exp2f(s[2 * tp + e / 4][e % 4]);
                sum[e % 2] = tp == 0 && e < 2 ? p[e] : sum[e % 2] + p[e];
                if (dp) dsum = fmaf(p[e], dp[2 * tp + e / 4][e % 4], dsum);
            }
            pb[tp] = pack8(p);
        }
        return sum[0] + sum[1];
    };
    if (FIRST) raise(false);
    float sum = weights();
    if (!FIRST && __builtin_amdgcn_ballot_w64(sum > 256.0f) != 0) {
        const float alpha = __builtin_amdgcn_exp2f(-raise(true));
        l *= alpha;
        if (dp) *d *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) acc[dt] *= alpha;
        sum = weights();
    }
    l += sum;
    if (dp) *d += dsum;
}

// A direct load of 16 bytes per lane to 1024 consecutive bytes of LDS (l: the same for all lanes) that the compiler does
// not count: it would wait for all outstanding ones before the next LDS read, those of the buffer in flight among them.
// The caller waits (s_waitcnt vmcnt) before it reads the buffer, and calls lds_reads_done() before it refills one.
// M0 is declared as overwritten, so that the compiler keeps no value of its own there across the load (it warns that it does
// not restore the register, and need not).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds_untracked(const bf16_t *g, bf16_t *l)
{
    const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) bf16_t *)l);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(g) : "memory", "m0");
}

// Four bytes per lane to 256 consecutive bytes of LDS, likewise.
__device__ __forceinline__ void load4_to_lds_untracked(const float *g, float *l)
{
    const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)l);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(at), "v"(g) : "memory", "m0");
}

#pragma clang diagnostic pop

// The wavefront's own reads of LDS have arrived in its registers: the compiler places the waits for them by their uses, and
// does not know that a direct load is about to overwrite what they read.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace mfma
}  // namespace bra
