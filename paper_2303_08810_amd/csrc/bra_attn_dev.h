// Device-side pieces of the routed attention kernels that stream rows straight into LDS (internal).
#pragma once

#include "bra_mfma_dev.h"

#include <type_traits>

namespace bra {
namespace mfma {

// How far above the largest score a reference is put (in units of log2): a power of two that weights, denominators and sums carry without
// loss, so that a later score moves the reference only once it is about twice as far above the earlier maximum.  A first block's
// weights are at most 2^-8, later ones up to 2^8; what lies 2^118 below the maximum is lost instead of 2^126.
constexpr float kHeadroom = 8.0f;

// Softmax step for KT tiles of 16 keys x 16 queries of one head: scores
// s[t][j] = S^T[key 16 t + 4 g + j][query i] relative to the reference m (which entered the product as its accumulator
// input, so a score costs no subtraction), weights p = 2^s in the operand order of O^T += V^T P^T.  l: the lane's share of
// the denominator, a sum of the float32 weights (over its keys: the caller adds up the four lane groups at the end).
// That sum also decides when the reference has to move: only when a lane's weights of a block exceed 2^8 together, which
// needs no maximum and no exchange between lanes; the quotient O / l does not depend on it.  FIRST: the reference is
// kHeadroom above this block's maximum.  With dp (scores of the gradient in the same layout) also d: the lane's share of sum p dp.
template <bool FIRST, int KT, int NDT>
__device__ __forceinline__ void softmax_step(f32x4 (&s)[KT], float &m, float &l, f32x4 (&acc)[NDT], bf16x8 (&pb)[KT / 2],
                                             const f32x4 *dp = nullptr, float *d = nullptr)
{
    auto raise = [&](bool keep) {               // moves the reference kHeadroom above the largest score; returns by how much
        float mx = s[0][0];
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) mx = fmaxf(mx, s[t][j]);
        const float top = cross_row_max(mx), up = keep && !(top > 0.f) ? 0.f : top + kHeadroom;
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

// Rows 16 t + i of a buffer's map as operands: piece p (rows of 64 elements; their 16-byte pieces lie exchanged, piece c of
// row r at c ^ r % 8).
__device__ __forceinline__ bf16x8 row_operand(const bf16_t *T, int row, int piece)
{
    return *(const bf16x8 *)(T + row * 64 + 8 * (piece ^ (row % 8)));
}

// Columns col0 + i of rows row0 .. row0 + 31 (contraction slots in the accumulator order: 4 g .. 4 g + 3, then 16 further).
__device__ __forceinline__ bf16x8 column_operand(const bf16_t *T, int row0, int col0, int g, int i)
{
    u32x2 r[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int row = row0 + 16 * half + 4 * g + i / 4, piece = col0 / 8 + (i % 4) / 2;
        r[half] = __builtin_bit_cast(u32x2, lds_read_tr16(T + row * 64 + 8 * (piece ^ (row % 8)) + 4 * (i % 2)));
    }
    return __builtin_bit_cast(bf16x8, u32x4{r[0][0], r[0][1], r[1][0], r[1][1]});
}

// Address in LDS, as the direct loads take it; the same for all lanes.
__device__ __forceinline__ unsigned lds_address(const void *l)
{
    return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)l);
}

// A direct load of 16 bytes per lane to the 1024 consecutive bytes from LDS address `at` on that the compiler does
// not count: it would wait for all outstanding ones before the next LDS read, those of the buffer in flight among them.
// The caller waits (s_waitcnt vmcnt) before it reads the buffer, and calls lds_reads_done() before it refills one.
// M0 is declared as overwritten, so that the compiler keeps no value of its own there across the load (it warns that it does
// not restore the register, and need not).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds_untracked(const bf16_t *g, unsigned at)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(g) : "memory", "m0");
}

// The same from `offset` bytes behind a base that is the same for all lanes.
__device__ __forceinline__ void load_to_lds_untracked(const bf16_t *base, unsigned offset, unsigned at)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(at), "v"(offset), "s"(base) : "memory", "m0");
}

// Four bytes per lane to 256 consecutive bytes of LDS, likewise.
__device__ __forceinline__ void load4_to_lds_untracked(const float *g, unsigned at)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(at), "v"(g) : "memory", "m0");
}

#pragma clang diagnostic pop

// The wavefront's own reads of LDS have arrived in its registers: the compiler places the waits for them by their uses, and
// does not know that a direct load is about to overwrite what they read.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Rows of a list of regions (origin by origin, n slots each), as a thread meets them: U rows `apart` from each other, all of
// them `step` further on with every advance().  The region and the slot are kept and carried along, and two tables in LDS
// give the token: divisions by n and by the region's width for every row were half of the vector instructions of
// k_attn_rows, and a fifth of k_attn_gen's (8 x 32 x 32 x 768, 12 regions of 16 tokens: whole layer 111.6 -> 109.4 us; gradients
// 25 x 8 x 16 x 768, k = 36: 267 -> 258 us, 11 x 42 x 42 x 256, k = 6: 212 -> 209, 12 x 112 x 120 x 64, k = 1: 272 -> 267).
// Rows past the end of the list meet its last region.
template <int U>
struct RowWalk {
    int p[U], s[U], n, step_p, step_s;
    __device__ __forceinline__ void start(int row, int apart, int step, int n_, float n_inv)
    {
        n = n_;
        step_p = divide(step, n, n_inv);
        step_s = step - step_p * n;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            p[u] = divide(row + apart * u, n, n_inv);
            s[u] = row + apart * u - p[u] * n;
        }
    }
    __device__ __forceinline__ void advance()
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int up = s[u] + step_s, wrapped = up - n;
            p[u] += step_p + (wrapped >= 0 ? 1 : 0);
            s[u] = (int)min((unsigned)up, (unsigned)wrapped);
        }
    }
    __device__ __forceinline__ void retreat()
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int down = s[u] - step_s, wrapped = down + n;
            p[u] -= step_p + (down < 0 ? 1 : 0);
            s[u] = (int)min((unsigned)down, (unsigned)wrapped);
        }
    }
    __device__ __forceinline__ int token(int u, const int *origins, int last, const int *slots) const
    {
        return origins[min(p[u], last)] + slots[s[u]];
    }
};

// What the walk takes: a slot table of 4 KB at most, token numbers of 24 bits and byte offsets of 32 within an image.
constexpr int kWalkMaxSlots = 1024;
inline bool walk_ok(const Dims &D)
{
    return D.n <= kWalkMaxSlots && D.N < (1 << 24) && (long)D.N * D.C * 2 < (1L << 32);
}

// Byte offset of a token's row, `lane_bytes` within it.
__device__ __forceinline__ unsigned row_offset(int token, int C, unsigned lane_bytes) { return __umul24((unsigned)token, 2u * (unsigned)C) + lane_bytes; }

}  // namespace mfma
}  // namespace bra
