// LCE (Eq. 7: depth-wise 5 x 5 correlation, stride 1, zero padding 2) of one region and 64 channels of a bf16 map, inside a workgroup of
// four wavefronts that works on that region anyway: what it is added to is then rounded once and no map lies between two kernels.
//
// The region with a halo of 2 goes from memory straight into LDS, a token's 64 channels in 128 bytes; the transposing LDS read gives
// a lane four neighbouring columns of ONE channel, packed as the pairs that v_dot2_f32_bf16 takes, so that nothing is permuted but the odd
// pairs (one instruction each): 264 vector instructions and 16 LDS reads for 16 outputs of a lane (walk_tile in bra_lce_pairs.h, whose
// lanes load two channels of a token: 21 per output).  Pairs and taps are those of walk_tile, and so is what an infinity reaches.
// Pieces of 16 bytes are exchanged: piece p of a token in column x of the halo at p ^ 2 (x / 2 % 4).  The columns of a read, and those of the
// lane groups beside it, meet different banks then.
#pragma once

#include "bra_attn_dev.h"
#include "bra_lce_pairs.h"

namespace bra {
namespace lce {

// Items of 4 x 4 outputs; the halo is as wide and as high as whole items need.
struct RegionHalo {
    int quads, strips;                   // items side by side, above each other
    __host__ __device__ constexpr RegionHalo(int rh, int rw) : quads((rw + 3) / 4), strips((rh + 3) / 4) {}
    __host__ __device__ constexpr int items() const { return quads * strips; }
    __host__ __device__ constexpr int width() const { return 4 * quads + 4; }
    __host__ __device__ constexpr int tokens() const { return (4 * strips + 4) * width(); }
    // LDS in bytes: the halo, later the float32 results of n tokens
    __host__ __device__ constexpr int bytes(int n) const { return tokens() * 128 > 4 * n * 68 ? tokens() * 128 : 4 * n * 68; }
};

constexpr int kResultPitch = 68;         // floats per token of the results

alignas(16) static __device__ bf16_t zero_piece[8];      // what tokens beyond the map read (never written)

// Requests the halo of the region whose first token is (y0, x0).  map: the image's, at its first of 64 channels.  The caller waits.
__device__ __forceinline__ void request_halo(const RegionHalo &r, const bf16_t *map, const Dims &D, int y0, int x0, unsigned at, int wave, int lane)
{
    const int width = r.width();
    const float w_inv = 1.0f / (float)width;
    for (int u = wave; u < r.tokens() / 8; u += 4) {
        const int t = 8 * u + lane / 8, hy = mfma::divide(t, width, w_inv), hx = t - hy * width, y = y0 - 2 + hy, x = x0 - 2 + hx;
        const int piece = (lane % 8) ^ 2 * (hx / 2 % 4);
        const bool in = (unsigned)y < (unsigned)D.H && (unsigned)x < (unsigned)D.W;
        mfma::load_to_lds_untracked(in ? map + ((size_t)y * D.W + x) * D.C + 8 * piece : zero_piece, at + 1024 * u);
    }
}

// The taps of channel c (the lane's; a multiple of 64 channels) as operands, [ky][(w0,w1) | (w2,w3) | (0,w4)].  A channel's 25 lie in 13 words,
// from the middle of the first one on if c is odd.
template <bool REVERSED>
struct LaneTaps {
    unsigned raw[13];
    bool odd;
    __device__ __forceinline__ LaneTaps(const bf16_t *__restrict__ Wlce, int c) : odd(c % 2 != 0)
    {
        const unsigned *from = (const unsigned *)(Wlce + (size_t)c * 25 - (odd ? 1 : 0));
#pragma unroll
        for (int j = 0; j < 13; ++j) raw[j] = from[j];
    }
    __device__ __forceinline__ void operands(unsigned (&w)[5][3]) const
    {
        unsigned t[13];                  // taps (2 j, 2 j + 1)
#pragma unroll
        for (int j = 0; j < 13; ++j) t[j] = odd ? __builtin_amdgcn_alignbit(j < 12 ? raw[j + 1] : 0u, raw[j], 16) : raw[j];
        auto pair = [&](int j) { return j % 2 ? __builtin_amdgcn_alignbit(t[j / 2 + 1], t[j / 2], 16) : t[j / 2]; };   // taps (j, j + 1)
#pragma unroll
        for (int ky = 0; ky < 5; ++ky) {
            const int j = REVERSED ? 20 - 5 * ky : 5 * ky;
            if (REVERSED) {              // taps 24 - 5 ky - kx
                const unsigned a = pair(j + 3), c = pair(j + 1), e = j % 2 ? t[j / 2] >> 16 : t[j / 2];
                w[ky][0] = __builtin_amdgcn_alignbit(a, a, 16);
                w[ky][1] = __builtin_amdgcn_alignbit(c, c, 16);
                w[ky][2] = e << 16;
            } else {
                w[ky][0] = pair(j);
                w[ky][1] = pair(j + 2);
                w[ky][2] = j % 2 ? t[(j + 4) / 2] & 0xffff0000u : t[(j + 4) / 2] << 16;
            }
        }
    }
};

// Row y of an item's window (0 .. 7), as pairs of columns (j, j + 1), into the sums of the 4 x 4 outputs that it belongs to.
__device__ __forceinline__ void add_row(int y, const unsigned (&p)[7], const unsigned (&w)[5][3], float (&o)[4][4])
{
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (y < a || y > a + 4) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            o[a][c] = dot2(w[y - a][0], p[c], o[a][c]);
            o[a][c] = dot2(w[y - a][1], p[c + 2], o[a][c]);
            o[a][c] = dot2(w[y - a][2], p[c + 3], o[a][c]);
        }
    }
}

// Sums of the lane's channel: lane group q has items q, q + 4, .. , ROUNDS of them; o[round][row][column].
template <int ROUNDS>
__device__ __forceinline__ void halo_sums(const RegionHalo &r, const bf16_t *halo, const unsigned (&w)[5][3], int wave, int lane, float (&o)[ROUNDS][4][4])
{
    const int s = lane % 16, width = r.width();
#pragma unroll
    for (int round = 0; round < ROUNDS; ++round) {
        if (4 * round >= r.items()) break;
        const int item = min(4 * round + lane / 16, r.items() - 1), strip = item / r.quads, quad = item - strip * r.quads;
        const bf16_t *at[2];             // the item's columns 0 to 3 and 4 to 7
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int hx = 4 * (quad + half) + s / 4;
            at[half] = halo + (4 * strip * width + hx) * 64 + 8 * ((2 * wave + s % 4 / 2) ^ 2 * (hx / 2 % 4)) + 4 * (s % 2);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[round][a][c] = 0.f;
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            unsigned p[7];               // columns (j, j + 1)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const mfma::u32x2 v = __builtin_bit_cast(mfma::u32x2, mfma::lds_read_tr16(at[half] + y * width * 64));
                p[4 * half] = v[0];
                p[4 * half + 2] = v[1];
            }
#pragma unroll
            for (int j = 1; j < 7; j += 2) p[j] = __builtin_amdgcn_alignbit(p[j + 1], p[j - 1], 16);
            add_row(y, p, w, o[round]);
        }
    }
}

// Leaves them in LDS, row by token of the region, kResultPitch floats apart.
template <int ROUNDS>
__device__ __forceinline__ void park_sums(const RegionHalo &r, const Dims &D, float *to, int wave, int lane, const float (&o)[ROUNDS][4][4])
{
#pragma unroll
    for (int round = 0; round < ROUNDS; ++round) {
        const int item = 4 * round + lane / 16, strip = item / r.quads, quad = item - strip * r.quads;
        if (4 * round >= r.items()) break;
        if (item >= r.items()) continue;
        float *at = to + (4 * strip * D.rw + 4 * quad) * kResultPitch + 16 * wave + lane % 16;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (4 * strip + a < D.rh && 4 * quad + c < D.rw) at[(a * D.rw + c) * kResultPitch] = o[round][a][c];
    }
}

// A slice of 32 channels of a whole image in LDS, `pitch` elements per token: items of 4 x 4 outputs of 16 channels on 16 lanes, a wavefront has two
// items (`first`, the same for all its lanes, and the next one) of both halves of the channels.  Tokens outside the image read `zero` (16 bytes of zeros).
// The last ones of a side of 4 or more end with the image: outputs that they share with the ones before come out twice, the same.
struct SliceItem {
    int y0, x0, at;                      // first output; this lane's column of the window's first row
    int rows, columns;                   // how many of the first ones the items before have too
    bool mine, left, right;              // there is such an item; the column lies in the image, the one 4 further does

    __device__ __forceinline__ SliceItem(const Dims &D, int first, int items, int quads, float q_inv, int lane, int pitch)
    {
        const int s = lane % 16, m = first + lane / 32, item = min(m, items - 1), strip = mfma::fast_div(item, q_inv);
        mine = m < items;
        const int quad = item - strip * quads;
        y0 = max(min(4 * strip, D.H - 4), 0);
        x0 = max(min(4 * quad, D.W - 4), 0);
        rows = 4 * strip - y0;
        columns = 4 * quad - x0;
        const int xl = x0 - 2 + s / 4;
        left = xl >= 0 && xl < D.W;
        right = xl + 4 < D.W;
        at = ((y0 - 2) * D.W + xl) * pitch + 16 * (lane / 16 % 2) + 4 * (s % 4);
    }
    // Row y of the window (0 .. 7) as pairs of columns (j, j + 1) of the lane's channel.
    __device__ __forceinline__ void pairs(const bf16_t *slice, const bf16_t *zero, int y, const Dims &D, int pitch, unsigned (&p)[7]) const
    {
        const bool in = (unsigned)(y0 + y - 2) < (unsigned)D.H;
        const bf16_t *from = slice + at + y * D.W * pitch;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const mfma::u32x2 v = __builtin_bit_cast(mfma::u32x2, mfma::lds_read_tr16(in && (half ? right : left) ? from + 4 * half * pitch : zero));
            p[4 * half] = v[0];
            p[4 * half + 2] = v[1];
        }
#pragma unroll
        for (int j = 1; j < 7; j += 2) p[j] = __builtin_amdgcn_alignbit(p[j + 1], p[j - 1], 16);
    }
    // The 16 sums of the lane's channel.
    __device__ __forceinline__ void sums(const bf16_t *slice, const bf16_t *zero, const Dims &D, int pitch, const unsigned (&w)[5][3], float (&o)[4][4]) const
    {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[a][c] = 0.f;
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            unsigned p[7];
            pairs(slice, zero, y, D, pitch, p);
            add_row(y, p, w, o);
        }
    }
    // Tap gradients: the image's own V against the window in dO; acc[5 ky + kx] belongs to tap 24 - (5 ky + kx).  Tokens of V that the items before have are
    // zeros here: they meet what those meet, so that an infinity of dO reaches no other taps.  Sides of at least 4.
    __device__ __forceinline__ void taps(const bf16_t *dO, const bf16_t *V, const bf16_t *zero, const Dims &D, int pitch, float (&acc)[25]) const
    {
        const bool own = mine && (int)(threadIdx.x % 16 / 4) >= columns;
        mfma::u32x2 v[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
            v[a] = __builtin_bit_cast(mfma::u32x2, mfma::lds_read_tr16(own && a >= rows ? V + at + (2 + (2 + a) * D.W) * pitch : zero));
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            unsigned p[7];
            pairs(dO, zero, y, D, pitch, p);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                if (y < a || y > a + 4) continue;
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    acc[5 * (y - a) + j] = dot2(v[a][0], p[j], acc[5 * (y - a) + j]);
                    acc[5 * (y - a) + j] = dot2(v[a][1], p[j + 2], acc[5 * (y - a) + j]);
                }
            }
        }
    }
};

}  // namespace lce
}  // namespace bra
