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
#include "bra_lce_dev.h"

namespace bra {
namespace lce {

namespace {

using namespace mfma;

// A window row: pairs of columns (0,1), (2,3), (4,5) | (1,2), (3,4) per channel.
struct Row {
    unsigned even[2][3], odd[2][2];
};

// How a workgroup's 8 column-pair slots lie on a map: `pairs` of them side by side, `subs` strips above each other
// (narrow maps).
struct Tiling {
    int pairs, subs, xtiles, ytiles, height;
};

// GRAD = false: Out += LCE(In).
// GRAD = true:  Out += LCE^T(In) (taps reversed) and the tap gradients from the same window (see k_lce_grad in
//               bra_lce_dev.h for the identities): (V left, V right) against the window's pairs (p, p + 1), 25 sums
//               per channel kept across the workgroup's tiles, Part[group][C][25] at the end.
template <bool GRAD>
__global__ __launch_bounds__(256) void k_lce_pairs(const bf16_t *__restrict__ In, const bf16_t *__restrict__ V,
                                                   const bf16_t *__restrict__ Wlce, bf16_t *__restrict__ Out, int ldo,
                                                   float *__restrict__ Part, Dims D, Tiling T, int cblocks, long tiles,
                                                   int tiles_per_wg)
{
    __shared__ __attribute__((aligned(16))) float red[GRAD ? 25 * 256 : 15 * 64];
    unsigned (*table)[3][64] = (unsigned (*)[3][64])red;      // [ky][(w0,w1) | (w2,w3) | (0,w4)][channel]
    const int block = mfma::swizzled_block(), cb = block % cblocks, c0 = 64 * cb, grp = block / cblocks;
    const long first = (long)grp * tiles_per_wg, last = min(tiles, first + tiles_per_wg);
    if (first >= tiles) return;
    const int cp = threadIdx.x % 32, slot = threadIdx.x / 32;
    for (int e = threadIdx.x; e < 5 * 64; e += 256) {
        const int ch = e % 64, ky = e / 64;
        unsigned t[5];
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
            const int tap = 5 * ky + kx;
            t[kx] = c0 + ch < D.C ? Wlce[(size_t)(c0 + ch) * 25 + (GRAD ? 24 - tap : tap)] : 0;
        }
        table[ky][0][ch] = t[0] | t[1] << 16;
        table[ky][1][ch] = t[2] | t[3] << 16;
        table[ky][2][ch] = t[4] << 16;
    }
    __syncthreads();
    const bool live = c0 + 2 * cp < D.C;
    const int cl = live ? 2 * cp : 0;
    u32x2 w[5][3];
#pragma unroll
    for (int ky = 0; ky < 5; ++ky)
#pragma unroll
        for (int t = 0; t < 3; ++t) w[ky][t] = *(const u32x2 *)&table[ky][t][cl];
    float acc[GRAD ? 25 : 1][2];
#pragma unroll
    for (int t = 0; t < (GRAD ? 25 : 1); ++t) acc[t][0] = acc[t][1] = 0.f;
    if (GRAD) __syncthreads();

    const int px = slot % T.pairs, sub = slot / T.pairs;
    for (long tile = first; tile < last; ++tile) {
        const int yt = (int)(tile / T.xtiles % T.ytiles), ybase = yt * T.subs * T.height;
        const int x0 = 2 * ((int)(tile % T.xtiles) * T.pairs + px), y0 = ybase + sub * T.height;
        const size_t b = tile / ((long)T.xtiles * T.ytiles);
        if (sub >= T.subs || x0 >= D.W || y0 >= D.H) continue;
        const int y1 = min(y0 + T.height, D.H), ytop = max(ybase - 2, 0);
        const bool right = x0 + 1 < D.W;
        // bases are the same for all lanes, lane offsets 32-bit from the tile's first row
        const char *ibase = (const char *)(In + (b * D.N + (size_t)ytop * D.W) * D.C + c0);
        const char *vbase = GRAD ? (const char *)(V + (b * D.N + (size_t)ytop * D.W) * D.C + c0) : nullptr;
        char *obase = (char *)(Out + (b * D.N + (size_t)ytop * D.W) * ldo + c0);
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
                nd[j] = *(const unsigned *)(obase + (yc * orow + oo[j]));
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
                float o[2][2] = {{bf16_lo(nd[0]), bf16_hi(nd[0])}, {bf16_lo(nd[1]), bf16_hi(nd[1])}};   // [column][channel]
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
                    char *row = obase + (unsigned)(y - ytop) * orow;
                    *(unsigned *)(row + oo[0]) = mfma::pack_bf16(o[0][0], o[0][1]);
                    if (right) *(unsigned *)(row + oo[1]) = mfma::pack_bf16(o[1][0], o[1][1]);
                }
            }
        }
    }
    if (!GRAD) return;
    // the 8 slots' sums of a channel through LDS, added in a fixed order
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < (GRAD ? 25 : 1); ++t) red[t * 256 + threadIdx.x] = acc[t][v];
        __syncthreads();
        for (int e = threadIdx.x; e < 25 * 32; e += 256) {
            const int t = e / 32, ch = c0 + 2 * (e % 32) + v;
            float s = 0.f;
            for (int k = 0; k < 8; ++k) s += red[t * 256 + k * 32 + e % 32];
            if (ch < D.C) Part[((size_t)grp * D.C + ch) * 25 + 24 - t] = s;
        }
    }
}

// Lane offsets are 32-bit: the rows of a tile (with the window, within the map) must span less than 2 GiB in either map.
bool offsets_fit(const Dims &D, const Tiling &T, int ldo)
{
    return (long)std::min(T.subs * T.height + 4, D.H) * D.W * std::max(D.C, ldo) * 2 < (1L << 31);
}

// Strips of 20 rows, or 10 or 5 where that leaves fewer than `want` tiles or the rows span too much.
Tiling tiling(const Dims &D, int ldo, long want, long &tiles)
{
    Tiling T;
    const int xp = (D.W + 1) / 2;
    T.pairs = xp < 8 ? xp : 8;
    T.xtiles = (xp + T.pairs - 1) / T.pairs;
    for (T.height = 20;; T.height /= 2) {
        const int strips = (D.H + T.height - 1) / T.height;
        T.subs = 8 / T.pairs < strips ? 8 / T.pairs : strips;
        T.ytiles = (strips + T.subs - 1) / T.subs;
        tiles = (long)D.B * T.xtiles * T.ytiles;
        if (T.height == 5 || (tiles >= want && offsets_fit(D, T, ldo))) return T;
    }
}

}  // namespace

// Maps so wide that not even strips of 5 rows fit (119 million values in a row) take the kernels of bra_lce_dev.h, whose
// addresses are 64-bit throughout.
int lce_add_bf16(const Dims &D, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, int ldo, int kernel_id, hipStream_t st)
{
    const int cblocks = (D.C + 63) / 64;
    long tiles;
    const Tiling T = tiling(D, ldo, 1536 / cblocks, tiles);
    const long blocks = tiles * cblocks;
    if (!offsets_fit(D, T, ldo)) return launch_lce<bf16_t, bf16_t>(D, V, D.C, Wlce, O, ldo, kernel_id, st);
    if (D.C % 2 || ldo % 2 || blocks > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_pairs<false>, dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, st, V, (const bf16_t *)nullptr,
                       Wlce, O, ldo, (float *)nullptr, D, T, cblocks, tiles, 1);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

namespace {

// About 768 workgroups (three per compute unit), each with the tiles of one group.
constexpr int kGradSlots = 768;

Tiling grad_plan(const Dims &D, int lddv, long &tiles, int &per_wg, int &groups)
{
    const int cblocks = (D.C + 63) / 64;
    const long want = std::max(1, kGradSlots / cblocks);
    const Tiling T = tiling(D, lddv, want, tiles);
    per_wg = (int)((tiles + want - 1) / want);
    groups = (int)((tiles + per_wg - 1) / per_wg);
    return T;
}

LcePlan wide_grad_plan(const Dims &D) { return lce_plan(D, kGradSlots, 8); }      // 8 columns per workgroup: two channels per thread

}  // namespace

int lce_grad_groups_bf16(const Dims &D, int lddv)
{
    long tiles;
    int per_wg, groups;
    return offsets_fit(D, grad_plan(D, lddv, tiles, per_wg, groups), lddv) ? groups : wide_grad_plan(D).groups;
}

int lce_grad_bf16(const Dims &D, const bf16_t *dO, const bf16_t *V, const bf16_t *Wlce, bf16_t *dV, int lddv, float *Part,
                  int kernel_id, hipStream_t st)
{
    const int cblocks = (D.C + 63) / 64;
    long tiles;
    int per_wg, groups;
    const Tiling T = grad_plan(D, lddv, tiles, per_wg, groups);
    if (D.C % 2 || lddv % 2) return BRA_ERR_UNSUPPORTED;
    if (!offsets_fit(D, T, lddv)) {
        ProfScope ps(st, kernel_id);
        return launch_lce_grad<bf16_t, bf16_t>(D, wide_grad_plan(D), dO, V, D.C, Wlce, dV, lddv, Part, st);
    }
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_lce_pairs<true>, dim3((unsigned)((groups * cblocks + 7) / 8 * 8)), dim3(256), 0, st, dO, V, Wlce, dV,
                       lddv, Part, D, T, cblocks, tiles, per_wg);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace lce
}  // namespace bra
