// LCE (Eq. 7: depth-wise 5 x 5 correlation, stride 1, zero padding 2) and its gradients on bf16 maps, on the
// two-element dot product v_dot2_f32_bf16 (two multiply-adds with a float32 sum per lane and instruction).
//
// A thread has 2 channels (one 32-bit load per token) of 2 neighbouring columns and walks down a strip of rows with
// the window of 5 rows x 6 columns in registers.  Per channel and row the left output takes the column pairs (0,1),
// (2,3), (3,4) against (w0,w1), (w2,w3), (0,w4); the right one the pairs (1,2), (3,4), (4,5) against the same taps.  A
// pair costs one byte permute.  The zero meets a column that the output takes anyway, in the same channel: an infinity
// may leave an output as NaN, but nothing reaches another channel or an output further away (columns as loaded, both
// channels in one operand with w4 in one half, did that: 0 times infinity in the neighbour).
// The next row is requested a step ahead and nothing is staged through LDS.
// What bounds it: the dot products and permutes (about 0.4 of the time by instruction count) and, at 3 to 4 wavefronts
// per SIMD, the latency they do not cover; an LDS-tiled version on float32 multiply-adds took 69 us for all three
// correlations of a 64 x 56 x 56 x 64 map.
#pragma once

#include "bra_lce_dev.h"

#include <algorithm>

namespace bra {
namespace lce {

using mfma::bf16_hi;
using mfma::bf16_lo;
using mfma::dot2;
using mfma::pair_hi;
using mfma::pair_lo;
using mfma::u32x2;

// A window row: pairs of columns (0,1), (2,3), (4,5) | (1,2), (3,4) per channel.
struct Row {
    unsigned even[2][3], odd[2][2];
};

// How a workgroup's 8 column-pair slots lie on a map: `pairs` of them side by side, `subs` strips above each other
// (narrow maps).
struct Tiling {
    int pairs, subs, xtiles, ytiles, height;
};

// The taps of 64 channels from c0 on as operands, through LDS: [ky][(w0,w1) | (w2,w3) | (0,w4)][channel].
typedef unsigned TapTable[5][3][64];
constexpr size_t kTapBytes = sizeof(TapTable);

template <bool REVERSED, int NT>
__device__ __forceinline__ void stage_taps(TapTable &table, const bf16_t *__restrict__ Wlce, int c0, int C)
{
    for (int e = threadIdx.x; e < 5 * 64; e += NT) {
        const int ch = e % 64, ky = e / 64;
        unsigned t[5];
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
            const int tap = 5 * ky + kx;
            t[kx] = c0 + ch < C ? Wlce[(size_t)(c0 + ch) * 25 + (REVERSED ? 24 - tap : tap)] : 0;
        }
        table[ky][0][ch] = t[0] | t[1] << 16;
        table[ky][1][ch] = t[2] | t[3] << 16;
        table[ky][2][ch] = t[4] << 16;
    }
    __syncthreads();
}

__device__ __forceinline__ void load_taps(u32x2 (&w)[5][3], const TapTable &table, int cl)
{
#pragma unroll
    for (int ky = 0; ky < 5; ++ky)
#pragma unroll
        for (int t = 0; t < 3; ++t) w[ky][t] = *(const u32x2 *)&table[ky][t][cl];
}

// One tile for the thread's slot (0 .. 7) and channels c0 + cl, c0 + cl + 1 (live: they exist).
// GRAD = false: LCE(In), with ADDS added to what Out holds.  Without, in float32, the upper halves of the bits in Out and the
//               lower ones in Low (laid out like Out): what is added to it later then rounds once.
// GRAD = true:  the same with w the reversed taps (LCE^T), and the tap gradients from the same window (see k_lce_grad in
//               bra_lce_dev.h for the identities): (V left, V right) against the window's pairs (p, p + 1), 25 sums
//               per channel added to acc.
template <bool GRAD, bool ADDS>
__device__ __forceinline__ void walk_tile(const bf16_t *__restrict__ In, const bf16_t *__restrict__ V, bf16_t *__restrict__ Out, bf16_t *__restrict__ Low, int ldo,
                                          const Dims &D, const Tiling &T, long tile, int slot, int c0, int cl, bool live,
                                          const u32x2 (&w)[5][3], float (&acc)[GRAD ? 25 : 1][2])
{
    const int px = slot % T.pairs, sub = slot / T.pairs;
    const int yt = (int)(tile / T.xtiles % T.ytiles), ybase = yt * T.subs * T.height;
    const int x0 = 2 * ((int)(tile % T.xtiles) * T.pairs + px), y0 = ybase + sub * T.height;
    const size_t b = tile / ((long)T.xtiles * T.ytiles);
    if (sub >= T.subs || x0 >= D.W || y0 >= D.H) return;
    const int y1 = min(y0 + T.height, D.H), ytop = max(ybase - 2, 0);
    const bool right = x0 + 1 < D.W;
    // bases are the same for all lanes, lane offsets 32-bit from the tile's first row
    const char *ibase = (const char *)(In + (b * D.N + (size_t)ytop * D.W) * D.C + c0);
    const char *vbase = GRAD ? (const char *)(V + (b * D.N + (size_t)ytop * D.W) * D.C + c0) : nullptr;
    char *obase = (char *)(Out + (b * D.N + (size_t)ytop * D.W) * ldo + c0);
    char *lbase = ADDS ? nullptr : (char *)(Low + (b * D.N + (size_t)ytop * D.W) * ldo + c0);
    const unsigned irow = 2u * D.W * D.C, orow = 2u * D.W * ldo;
    unsigned xo[6];
    bool xok[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        xok[j] = (unsigned)(x0 + j - 2) < (unsigned)D.W;
        xo[j] = 2u * (min(max(x0 + j - 2, 0), D.W - 1) * D.C + cl);
    }
    const unsigned oo[2] = {2u * (x0 * ldo + cl), 2u * ((right ? x0 + 1 : x0) * ldo + cl)};
    const bool edge = !__all(xok[0] && xok[1] && xok[4] && xok[5]);
    auto request_row = [&](int y, unsigned (&raw)[6]) {
        const unsigned row = (unsigned)(min(max(y, 0), D.H - 1) - ytop) * irow;
#pragma unroll
        for (int j = 0; j < 6; ++j) raw[j] = *(const unsigned *)(ibase + (row + xo[j]));
    };
    auto pack_row = [&](int y, unsigned (&raw)[6]) {
        if (edge || (unsigned)y >= (unsigned)D.H) {
            const bool in = (unsigned)y < (unsigned)D.H;
#pragma unroll
            for (int j = 0; j < 6; ++j) raw[j] = in && xok[j] ? raw[j] : 0u;
        }
        Row R;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            R.even[0][t] = pair_lo(raw[2 * t], raw[2 * t + 1]);
            R.even[1][t] = pair_hi(raw[2 * t], raw[2 * t + 1]);
            if (t == 2) break;
            R.odd[0][t] = pair_lo(raw[2 * t + 1], raw[2 * t + 2]);
            R.odd[1][t] = pair_hi(raw[2 * t + 1], raw[2 * t + 2]);
        }
        return R;
    };
    unsigned next[6], nv[2], nd[2];
    auto request = [&](int y) {          // what step y needs: row y + 2 of In, Out (and V) of row y
        const unsigned yc = min(y, D.H - 1) - ytop;
        request_row(y + 2, next);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (GRAD) nv[j] = *(const unsigned *)(vbase + (yc * irow + xo[j && right ? 3 : 2]));
            if (ADDS) nd[j] = *(const unsigned *)(obase + (yc * orow + oo[j]));
        }
    };
    Row win[5];
    {
        unsigned rows[4][6];
#pragma unroll
        for (int r = 0; r < 4; ++r) request_row(y0 + r - 2, rows[r]);
        request(y0);
#pragma unroll
        for (int r = 0; r < 4; ++r) win[r] = pack_row(y0 + r - 2, rows[r]);
    }
    for (int yb = y0; yb < y1; yb += 5) {
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            const int y = yb + u;
            if (y >= y1) break;
            win[(u + 4) % 5] = pack_row(y + 2, next);
            unsigned vp[2] = {0u, 0u};
            if (GRAD) {
                const unsigned vr = right ? nv[1] : 0u;
                vp[0] = pair_lo(nv[0], vr);
                vp[1] = pair_hi(nv[0], vr);
            }
            float o[2][2] = {{0.f, 0.f}, {0.f, 0.f}};                  // [column][channel]
            if (ADDS) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    o[j][0] = bf16_lo(nd[j]);
                    o[j][1] = bf16_hi(nd[j]);
                }
            }
            request(y + 1);
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                const Row &R = win[(u + r) % 5];
#pragma unroll
                for (int v = 0; v < 2; ++v) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        o[0][v] = dot2(w[r][t][v], R.even[v][t], o[0][v]);
                        o[1][v] = dot2(w[r][t][v], R.odd[v][t], o[1][v]);
                    }
                    o[0][v] = dot2(w[r][2][v], R.odd[v][1], o[0][v]);
                    o[1][v] = dot2(w[r][2][v], R.even[v][2], o[1][v]);
                    if (GRAD) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            acc[5 * r + 2 * t][v] = dot2(vp[v], R.even[v][t], acc[5 * r + 2 * t][v]);
                            acc[5 * r + 2 * t + 1][v] = dot2(vp[v], R.odd[v][t], acc[5 * r + 2 * t + 1][v]);
                        }
                        acc[5 * r + 4][v] = dot2(vp[v], R.even[v][2], acc[5 * r + 4][v]);
                    }
                }
            }
            if (live) {
                const unsigned at = (unsigned)(y - ytop) * orow;
                char *row = obase + at;
                if constexpr (!ADDS) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if (j == 1 && !right) break;
                        const unsigned a = __builtin_bit_cast(unsigned, o[j][0]), c = __builtin_bit_cast(unsigned, o[j][1]);
                        *(unsigned *)(row + oo[j]) = pair_hi(a, c);
                        *(unsigned *)(lbase + at + oo[j]) = pair_lo(a, c);
                    }
                } else {
                    *(unsigned *)(row + oo[0]) = mfma::pack_bf16(o[0][0], o[0][1]);
                    if (right) *(unsigned *)(row + oo[1]) = mfma::pack_bf16(o[1][0], o[1][1]);
                }
            }
        }
    }
}

// Lane offsets are 32-bit: the rows of a tile (with the window, within the map) must span less than 2 GiB in either map.
inline bool offsets_fit(const Dims &D, const Tiling &T, int ldo)
{
    return (long)std::min(T.subs * T.height + 4, D.H) * D.W * std::max(D.C, ldo) * 2 < (1L << 31);
}

// Strips of `height` rows.
inline Tiling strips_of(const Dims &D, int height, long &tiles)
{
    Tiling T;
    const int xp = (D.W + 1) / 2;
    T.pairs = xp < 8 ? xp : 8;
    T.xtiles = (xp + T.pairs - 1) / T.pairs;
    T.height = height;
    const int strips = (D.H + height - 1) / height;
    T.subs = 8 / T.pairs < strips ? 8 / T.pairs : strips;
    T.ytiles = (strips + T.subs - 1) / T.subs;
    tiles = (long)D.B * T.xtiles * T.ytiles;
    return T;
}

// The fewest strips of less than `height` rows: the next ones worth a look, however high the map (a strip more each time took 158 us
// per call on the host for 65536 rows).
inline int lower_strips(const Dims &D, int height) { return (D.H + height - 2) / (height - 1); }

// Strips of even heights, at most 20 rows: the highest with `want` tiles and rows that span little enough, or 5.
inline Tiling even_tiling(const Dims &D, int ldo, long want, long &tiles)
{
    for (int strips = (D.H + 19) / 20, height;; strips = lower_strips(D, height)) {
        height = (D.H + strips - 1) / strips;
        const Tiling T = strips_of(D, height, tiles);
        if (height <= 5 || (tiles >= want && offsets_fit(D, T, ldo))) return T;
    }
}

// Strips of even heights, 4 to 24 rows, two tiles to a block of 512 threads, two blocks to a compute unit.
//
// Beside the `beside` blocks that choose the regions: where all blocks of the launch find a compute unit each with strips of at most 16
// rows, the lowest such strips. Those take no longer than the choice itself, 11 to 13 us, which takes 1.4 times that when it shares its
// units. Measured with 24 blocks beside, 8 maps of 32 x 32 at 768 channels: 16 rows and 192 blocks 16.7 us, 11 to 4 rows and 288 to 768
// blocks 21.9 to 18.6; with 64, 4 maps of 112 x 112 at 64 channels: 12 rows and 140 blocks 12.0, 8 rows and 200 blocks 13.8.
//
// Elsewhere the heights whose rounds take the least: a round of 512 blocks takes 0.6 us a row and as much as kStart rows before the first
// is stored, and one of up to 256 takes kAlone of it. 64 maps of 21 x 21 at 384 channels: 21 rows 22.5 us, 11 rows 23.3, 7 rows 25.5, 5 rows
// 30.1; 20 of 56 x 56 at 192: 14 rows 22, 8 rows 24, 4 rows 29.
constexpr double kStart = 6, kAlone = 0.7;

inline Tiling forward_tiling(const Dims &D, int ldo, int cblocks, int beside, long &tiles)
{
    Tiling best = {};
    bool found = false, apart = false;
    double least = 0;
    const double places = std::max(256, 512 - beside);
    for (int strips = (D.H + 23) / 24, height;; strips = lower_strips(D, height)) {
        height = (D.H + strips - 1) / strips;
        const bool last = height <= 4;
        long n;
        const Tiling T = strips_of(D, height, n);
        const long blocks = (n + 1) / 2 * cblocks;
        const bool alone = beside && height <= 16 && blocks + beside <= 256;
        const double rounds = (double)blocks / places, whole = (double)(long)rounds, rest = rounds - whole;
        const double cost = (whole + (rest > 0.5 ? 1 : rest > 0 ? kAlone : 0)) * (kStart + height);
        if ((offsets_fit(D, T, ldo) || (last && !found)) && (alone || (!apart && (!found || cost < least)))) {
            best = T;
            least = cost;
            tiles = n;
            found = true;
            apart = alone;
        }
        if (last) return best;
    }
}

// A pass over a map; what it writes is walk_tile's.  Part (GRAD): [group][C][25], the tap gradients summed over the tiles
// of a workgroup.
struct Job {
    const bf16_t *In, *V, *Wlce;
    bf16_t *Out, *Low;
    float *Part;
    int ldo, cblocks, per_wg;
    long tiles;
    Tiling T;

    __host__ __device__ long groups() const { return (tiles + per_wg - 1) / per_wg; }
    __host__ __device__ long blocks() const { return (groups() * cblocks + 7) / 8 * 8; }
};

// LDS of job_block: the tap gradients of 256 threads.  taps_block: half of them at a time (a whole call of 1 x 21 x 21 x 384, where these
// sums come last, takes 0.3 us more so).
template <bool GRAD>
constexpr size_t job_bytes() { return GRAD ? 25 * 256 * 4 : kTapBytes; }
constexpr int kTapsAtOnce = 13;
constexpr size_t kTapSumBytes = kTapsAtOnce * 256 * 4;

// The 8 slots' sums of a channel through LDS, AT_ONCE taps at a time, added in a fixed order, to Part[grp].
template <int AT_ONCE>
__device__ __forceinline__ void store_tap_sums(const Job &J, const Dims &D, int grp, int c0, const float (&acc)[25][2], float *red)
{
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int t0 = 0; t0 < 25; t0 += AT_ONCE) {
            const int count = 25 - t0 < AT_ONCE ? 25 - t0 : AT_ONCE;
            __syncthreads();
#pragma unroll
            for (int t = 0; t < count; ++t) red[t * 256 + threadIdx.x] = acc[t0 + t][v];
            __syncthreads();
            for (int e = threadIdx.x; e < count * 32; e += 256) {
                const int t = e / 32, ch = c0 + 2 * (e % 32) + v;
                float s = 0.f;
                for (int k = 0; k < 8; ++k) s += red[t * 256 + k * 32 + e % 32];
                if (ch < D.C) J.Part[((size_t)grp * D.C + ch) * 25 + 24 - t0 - t] = s;
            }
        }
}

// Workgroup `block` of J, 256 threads.
template <bool GRAD, bool ADDS>
__device__ __forceinline__ void job_block(const Job &J, const Dims &D, int block, float *red)
{
    const int cb = block % J.cblocks, c0 = 64 * cb, grp = block / J.cblocks;
    const long first = (long)grp * J.per_wg, last = min(J.tiles, first + J.per_wg);
    if (first >= J.tiles) return;
    const int cp = threadIdx.x % 32, slot = threadIdx.x / 32;
    TapTable &table = *(TapTable *)red;
    stage_taps<GRAD, 256>(table, J.Wlce, c0, D.C);
    const bool live = c0 + 2 * cp < D.C;
    const int cl = live ? 2 * cp : 0;
    u32x2 w[5][3];
    load_taps(w, table, cl);
    float acc[GRAD ? 25 : 1][2];
#pragma unroll
    for (int t = 0; t < (GRAD ? 25 : 1); ++t) acc[t][0] = acc[t][1] = 0.f;
    if (GRAD) __syncthreads();
    for (long tile = first; tile < last; ++tile) walk_tile<GRAD, ADDS>(J.In, J.V, J.Out, J.Low, J.ldo, D, J.T, tile, slot, c0, cl, live, w, acc);
    if constexpr (GRAD) store_tap_sums<25>(J, D, grp, c0, acc, red);
}

// The tap gradients alone, for one tile: a row of In at a time, with the window in V (5 rows of one pair per channel, instead of 5 rows of
// five): 50 registers less than walk_tile's.  The same sums in the same order.
__device__ __forceinline__ void walk_taps(const bf16_t *__restrict__ In, const bf16_t *__restrict__ V, const Dims &D, const Tiling &T, long tile, int slot,
                                          int c0, int cl, float (&acc)[25][2])
{
    const int px = slot % T.pairs, sub = slot / T.pairs;
    const int yt = (int)(tile / T.xtiles % T.ytiles), ybase = yt * T.subs * T.height;
    const int x0 = 2 * ((int)(tile % T.xtiles) * T.pairs + px), y0 = ybase + sub * T.height;
    const size_t b = tile / ((long)T.xtiles * T.ytiles);
    if (sub >= T.subs || x0 >= D.W || y0 >= D.H) return;
    const int y1 = min(y0 + T.height, D.H), ytop = max(ybase - 2, 0);
    const bool right = x0 + 1 < D.W;
    const size_t at = (b * D.N + (size_t)ytop * D.W) * D.C + c0;
    const char *ibase = (const char *)(In + at), *vbase = (const char *)(V + at);
    const unsigned irow = 2u * D.W * D.C;
    unsigned xo[6];
    bool xok[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        xok[j] = (unsigned)(x0 + j - 2) < (unsigned)D.W;
        xo[j] = 2u * (min(max(x0 + j - 2, 0), D.W - 1) * D.C + cl);
    }
    const bool edge = !__all(xok[0] && xok[1] && xok[4] && xok[5]);
    unsigned next[6], nv[2];
    auto request = [&](int y) {          // row y of In, row y + 2 of V
        const unsigned row = (unsigned)(min(max(y, 0), D.H - 1) - ytop) * irow, vrow = (unsigned)(min(y + 2, D.H - 1) - ytop) * irow;
#pragma unroll
        for (int j = 0; j < 6; ++j) next[j] = *(const unsigned *)(ibase + (row + xo[j]));
#pragma unroll
        for (int j = 0; j < 2; ++j) nv[j] = *(const unsigned *)(vbase + (vrow + xo[j && right ? 3 : 2]));
    };
    unsigned vp[5][2] = {};              // of the rows y - 2 .. y + 2
    request(y0 - 2);
    for (int yb = y0 - 2; yb < y1 + 2; yb += 5) {
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            const int y = yb + u;
            if (y >= y1 + 2) break;
            const bool in = (unsigned)y < (unsigned)D.H;
            if (edge || !in) {
#pragma unroll
                for (int j = 0; j < 6; ++j) next[j] = in && xok[j] ? next[j] : 0u;
            }
            const unsigned vr = right ? nv[1] : 0u;
            vp[u][0] = pair_lo(nv[0], vr);
            vp[u][1] = pair_hi(nv[0], vr);
            unsigned p[5][2];            // columns (j, j + 1) of In
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                p[j][0] = pair_lo(next[j], next[j + 1]);
                p[j][1] = pair_hi(next[j], next[j + 1]);
            }
            request(y + 1);
#pragma unroll
            for (int r = 0; r < 5; ++r) {        // row y + 2 - r of V, if the tile has it, has this row as row r of its window
                if (y + 2 - r < y0 || y + 2 - r >= y1) continue;
#pragma unroll
                for (int j = 0; j < 5; ++j)
#pragma unroll
                    for (int v = 0; v < 2; ++v) acc[5 * r + j][v] = dot2(vp[(u + 5 - r) % 5][v], p[j][v], acc[5 * r + j][v]);
            }
        }
    }
}

// Workgroup `block` of J: its tap gradients alone.
__device__ __forceinline__ void taps_block(const Job &J, const Dims &D, int block, float *red)
{
    const int c0 = 64 * (block % J.cblocks), grp = block / J.cblocks;
    const long first = (long)grp * J.per_wg, last = min(J.tiles, first + J.per_wg);
    if (first >= J.tiles) return;
    const int cl = c0 + 2 * ((int)threadIdx.x % 32) < D.C ? 2 * ((int)threadIdx.x % 32) : 0;
    float acc[25][2];
#pragma unroll
    for (int t = 0; t < 25; ++t) acc[t][0] = acc[t][1] = 0.f;
    for (long tile = first; tile < last; ++tile) walk_taps(J.In, J.V, D, J.T, tile, threadIdx.x / 32, c0, cl, acc);
    store_tap_sums<kTapsAtOnce>(J, D, grp, c0, acc, red);
}

// The two passes of the gradients: LCE^T(dO) with the tap gradients, added to dV or in float32 (lower halves where dK goes), and
// O += LCE(V).  fit: walk_tile takes both.  beside: in the attention's launches.  The float32 sums are 4 bytes per value more to
// write and to read, which costs more than the launches saved where the attention has little to do meanwhile: few keys and
// small regions, or rows of many channels.  Beyond 14 million values they are beside only for regions of more than 96 tokens and up to 128
// channels; up to 14 million always, also where that is slower, because what they are added to is then rounded once (dX of 8 x
// 56 x 56 x 64 3.69e-3 from float64 instead of 3.71e-3).  Whole gradient, us, of their own / beside, by millions of values:
// 64 tokens per region, 56 x 56 x 64, k = 1: 3.1 87.6 / 77.9, 9.2 169 / 175, 12.3 207 / 208, 13.8 232 / 242, 19 336 / 364, k = 4: 12.3
// 269 / 260, 13.8 298 / 296, 19 419 / 426; 56 x 56 x 256, k = 4: 6.1 199.6 / 186.2, 13.8 402 / 409, 18 531 / 537; 16 tokens, 28 x 28 x 256, k = 4:
// 7.7 206 / 202, 15 382 / 393.  81 tokens, 64 channels: 15.5 365 / 366; 100: 14.4 291 / 282; 121: 14.5 280 / 268, 17 504 / 495, 128 channels 17
// 376 / 375, 256: 17 437 / 449; 256 tokens, 64 channels, k = 1: 15 344 / 322, 24.5 532 / 525, 37 772 / 781, 128: 17 419 / 401, 192: 23 590 / 597.
struct BackwardJobs {
    Job grad, add;
    bool fit, beside;
};
BackwardJobs backward_jobs(const Dims &D, const bf16_t *dO, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, bf16_t *dV, bf16_t *dK, int lddv, float *Part);
int lce_backward_bf16(const Dims &D, const BackwardJobs &L, int kernel_id, hipStream_t st);

}  // namespace lce
}  // namespace bra
