// The depth-wise 5 x 5 correlation (LCE, Eq. 7) and its gradients over whole token maps (internal): threads
// walk down image columns with the window in registers; no halo tiles, no barriers between rows.  The
// kernels of this header take float32 or bf16 maps and any channel count; bra_lce.hip has the bf16 ones for
// even channel counts.
#pragma once

#include "bra_mfma_dev.h"

#include <algorithm>
#include <type_traits>

namespace bra {
namespace lce {

using mfma::bf16_hi;
using mfma::bf16_lo;
using mfma::f32x2;

// VW (2 or 1) consecutive channels as float32.
template <int VW>
struct Channels {
    float v[VW];
};
template <int VW>
__device__ __forceinline__ Channels<VW> load_channels(const float *p)
{
    Channels<VW> r;
    if (VW == 2) {
        const f32x2 t = *(const f32x2 *)p;
        r.v[0] = t[0];
        r.v[VW - 1] = t[1];
    } else {
        r.v[0] = *p;
    }
    return r;
}
template <int VW>
__device__ __forceinline__ Channels<VW> load_channels(const bf16_t *p)
{
    Channels<VW> r;
    if (VW == 2) {
        const unsigned t = *(const unsigned *)p;
        r.v[0] = bf16_lo(t);
        r.v[VW - 1] = bf16_hi(t);
    } else {
        r.v[0] = bf16_to_f32(*p);
    }
    return r;
}
template <int VW>
__device__ __forceinline__ void store_channels(float *p, const Channels<VW> &r)
{
    if (VW == 2) *(f32x2 *)p = f32x2{r.v[0], r.v[VW - 1]};
    else *p = r.v[0];
}
template <int VW>
__device__ __forceinline__ void store_channels(bf16_t *p, const Channels<VW> &r)
{
    if (VW == 2) *(unsigned *)p = mfma::pack_bf16(r.v[0], r.v[VW - 1]);
    else *p = f32_to_bf16(r.v[0]);
}

// Workgroups of a pass beside those of another kernel, in front of them or behind: true for the `beside` ones of the pass.
// block: the number within its own kind.  (Evenly among the others, the two slow each other down: see launch_attn_bwd.)
__device__ __forceinline__ bool block_of_pass(int beside, bool front, int &block, int &blocks)
{
    const int others = (int)gridDim.x - beside, first = front ? 0 : others;
    const bool of_pass = (int)blockIdx.x >= first && (int)blockIdx.x < first + beside;
    block = (int)blockIdx.x - (of_pass ? first : front ? beside : 0);
    blocks = of_pass ? beside : others;
    return of_pass;
}

// The [C][25] taps, float32 or bf16.
struct Taps {
    const void *w;
    bool bf16;

    Taps() : w(nullptr), bf16(false) {}
    explicit Taps(const float *p) : w(p), bf16(false) {}
    explicit Taps(const bf16_t *p) : w(p), bf16(true) {}
};

// The taps of channels c0 .. c0 + 63 (those that exist) -> table[25][64], requested all at once.
template <int NT>
__device__ __forceinline__ void stage_taps(const Taps &taps, int c0, int C, float *table)
{
    constexpr int L = (25 * 64 + NT - 1) / NT;
    const int count = min(64, C - c0) * 25;
    float v[L];
    if (taps.bf16) {
#pragma unroll
        for (int u = 0; u < L; ++u) v[u] = bf16_to_f32(((const bf16_t *)taps.w)[(size_t)c0 * 25 + min((int)threadIdx.x + NT * u, count - 1)]);
    } else {
#pragma unroll
        for (int u = 0; u < L; ++u) v[u] = ((const float *)taps.w)[(size_t)c0 * 25 + min((int)threadIdx.x + NT * u, count - 1)];
    }
#pragma unroll
    for (int u = 0; u < L; ++u) {
        const int e = threadIdx.x + NT * u;
        if (e < count) table[e % 25 * 64 + e / 25] = v[u];
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Out[t][c] += sum_{ky,kx} w[c][ky][kx] In[t + (ky - 2, kx - 2)][c] over the H x W map (zero outside):
// LCE (Eq. 7).  Workgroup: 64 channels; a wavefront takes kLceRows rows of VW neighbouring pairs of columns, a thread VW (2 or
// 1) channels of one pair: an input row of 6 columns is read once and goes into the outputs it belongs to.  Image and rows
// are the same for all lanes, so that a load is a scalar row address and a 32-bit lane offset.  The taps pass through
// LDS once per workgroup: read per thread from the [C][25] tensor they would cost a cache line per lane.
// Bound by the FMAs and by the latency of the first of its eight rows; each further one is requested a row ahead.  16 x 56 x 56 x 64 float32 beside the routing: 11 us for
// both, 19 with one column per thread and addresses of its own for every load (k_lce_far; 122 registers for 84).
// Row pitches ldi, ldo.
constexpr int kLceRows = 4;

template <typename TM>
struct AddJob {
    const TM *In;
    Taps taps;
    TM *Out;
    int ldi, ldo, cblocks, blocks, groups;       // groups: of VW pairs of columns in a row
};

// Workgroup `block` of J, NT threads; table: [25][64].  ADDS = false: Out = LCE(In).  AHEAD: rows requested a row ahead.
template <int VW, bool ADDS, int NT, bool AHEAD = true, typename TM>
__device__ __forceinline__ void lce_block(const AddJob<TM> &J, const Dims &D, int block, float *table)
{
    constexpr int CPW = 64 / VW;
    const int cb = block % J.cblocks, c0 = 64 * cb, strips = (D.H + kLceRows - 1) / kLceRows;
    stage_taps<NT>(J.taps, c0, D.C, table);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, cl = lane % CPW * VW;
    const int q = block / J.cblocks * (NT / 64) + wave, gx = q % J.groups, y0 = q / J.groups % strips * kLceRows, b = q / (J.groups * strips);
    const int x = 2 * (gx * VW + lane / CPW);
    if (b >= D.B || x >= D.W || c0 + cl >= D.C) return;
    const bool right = x + 1 < D.W;
    unsigned xo[6];
    bool xok[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        xok[j] = (unsigned)(x + j - 2) < (unsigned)D.W;
        xo[j] = (unsigned)sizeof(TM) * (min(max(x + j - 2, 0), D.W - 1) * J.ldi + cl);
    }
    const bool edge = !__all(xok[0] && xok[1] && xok[4] && xok[5]);
    float w[25][VW];
#pragma unroll
    for (int t = 0; t < 25; ++t)
#pragma unroll
        for (int v = 0; v < VW; ++v) w[t][v] = table[64 * t + cl + v];
    Channels<VW> acc[kLceRows][2] = {};
    const char *img = (const char *)(J.In + (size_t)b * D.N * J.ldi + c0);
    const size_t pitch = sizeof(TM) * (size_t)D.W * J.ldi;
    Channels<VW> raw[2][6];
    auto request = [&](int dy) {                 // from a row of the map in any case
        const char *row = img + min(max(y0 + dy - 2, 0), D.H - 1) * pitch;
#pragma unroll
        for (int j = 0; j < 6; ++j) raw[dy % 2][j] = load_channels<VW>((const TM *)(row + xo[j]));
    };
    if (AHEAD) request(0);
#pragma unroll
    for (int dy = 0; dy < kLceRows + 4; ++dy) {
        const int y = y0 + dy - 2;
        if (AHEAD && dy + 1 < kLceRows + 4) request(dy + 1);
        if (y < 0 || y >= D.H) continue;
        if (!AHEAD) request(dy);
        Channels<VW> in[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) in[j] = raw[dy % 2][j];
        if (edge) {
#pragma unroll
            for (int j = 0; j < 6; ++j)
#pragma unroll
                for (int v = 0; v < VW; ++v) in[j].v[v] = xok[j] ? in[j].v[v] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < kLceRows; ++r) {
            const int ky = dy - r;
            if (ky < 0 || ky > 4) continue;
#pragma unroll
            for (int kx = 0; kx < 5; ++kx)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < VW; ++v) acc[r][j].v[v] = fmaf(w[5 * ky + kx][v], in[kx + j].v[v], acc[r][j].v[v]);
        }
    }
    char *out = (char *)(J.Out + ((size_t)b * D.N + (size_t)y0 * D.W) * J.ldo + c0);
    const unsigned oo = (unsigned)sizeof(TM) * (x * J.ldo + cl), ostep = (unsigned)sizeof(TM) * J.ldo;
#pragma unroll
    for (int r = 0; r < kLceRows; ++r) {
        if (y0 + r >= D.H) break;
        char *row = out + r * (sizeof(TM) * (size_t)D.W * J.ldo);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (j && !right) break;
            TM *at = (TM *)(row + (oo + j * ostep));
            Channels<VW> o = acc[r][j];
            if (ADDS) {
                const Channels<VW> there = load_channels<VW>(at);
#pragma unroll
                for (int v = 0; v < VW; ++v) o.v[v] += there.v[v];
            }
            store_channels<VW>(at, o);
        }
    }
}

// Not ahead with five workgroups per compute unit, by 13 registers: where four take a second round for what is left (layer with a given index, us, ahead / not: 32 x 28 x 28 x 160 bf16, 1176
// workgroups 68.9 / 66.6, 27 x 35 x 35 x 96, 1094 108.4 / 107.0; against that 784: 32 x 28 x 28 x 128 float32 70.0 / 70.7; 1536: 4 x 64 x 128 x 160 96.8 / 99.1; 98: 1 x 56 x 56 x 64 22.8 / 24.4).
template <typename TM, int VW, bool AHEAD>
__global__ __launch_bounds__(256, AHEAD ? 4 : 5) void k_lce(AddJob<TM> J, Dims D)
{
    __shared__ float table[25 * 64];
    lce_block<VW, true, 256, AHEAD>(J, D, mfma::swizzled_block(), table);
}

// The same for maps that k_lce's 32-bit offsets and numbers do not cover: a thread takes kLceRows rows of one column, all
// addresses 64-bit.
template <typename TM, int VW>
__global__ __launch_bounds__(256) void k_lce_far(const TM *__restrict__ In, int ldi, Taps source, TM *__restrict__ Out, int ldo,
                                                 Dims D, int cblocks)
{
    __shared__ float taps[25 * 64];
    constexpr int CPW = 64 / VW, COLS = 256 / CPW;
    const int block = mfma::swizzled_block(), cb = block % cblocks, c0 = 64 * cb, yb_n = (D.H + kLceRows - 1) / kLceRows;
    stage_taps<256>(source, c0, D.C, taps);
    const int cl = ((int)threadIdx.x % CPW) * VW, c = c0 + cl;
    const long q = (long)(block / cblocks) * COLS + threadIdx.x / CPW;
    if (q >= (long)D.B * yb_n * D.W || c >= D.C) return;
    const int x = (int)(q % D.W), y0 = (int)((q / D.W) % yb_n) * kLceRows;
    const size_t b = q / ((long)D.W * yb_n);
    const TM *img = In + b * D.N * ldi + c;
    TM *out = Out + (b * D.N + (size_t)y0 * D.W + x) * ldo + c;
    float w[25][VW];
#pragma unroll
    for (int t = 0; t < 25; ++t)
#pragma unroll
        for (int v = 0; v < VW; ++v) w[t][v] = taps[64 * t + cl + v];
    Channels<VW> acc[kLceRows];
#pragma unroll
    for (int r = 0; r < kLceRows; ++r)
#pragma unroll
        for (int v = 0; v < VW; ++v) acc[r].v[v] = 0.f;
#pragma unroll
    for (int dy = 0; dy < kLceRows + 4; ++dy) {
        const int y = y0 + dy - 2;
        const bool row_in = (unsigned)y < (unsigned)D.H;
        Channels<VW> in[5];
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
            const int xx = x + kx - 2;
            const bool ok = row_in && (unsigned)xx < (unsigned)D.W;
            in[kx] = load_channels<VW>(img + (size_t)(ok ? y * D.W + xx : 0) * ldi);
#pragma unroll
            for (int v = 0; v < VW; ++v) in[kx].v[v] = ok ? in[kx].v[v] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < kLceRows; ++r) {
            const int ky = dy - r;
            if (ky < 0 || ky > 4) continue;
#pragma unroll
            for (int kx = 0; kx < 5; ++kx)
#pragma unroll
                for (int v = 0; v < VW; ++v) acc[r].v[v] = fmaf(w[5 * ky + kx][v], in[kx].v[v], acc[r].v[v]);
        }
    }
#pragma unroll
    for (int r = 0; r < kLceRows; ++r) {
        if (y0 + r >= D.H) break;
        Channels<VW> o = load_channels<VW>(out + (size_t)r * D.W * ldo);
#pragma unroll
        for (int v = 0; v < VW; ++v) o.v[v] += acc[r].v[v];
        store_channels<VW>(out + (size_t)r * D.W * ldo, o);
    }
}

// blocks: a multiple of 8; 0 where offsets or numbers need more than 32 bits.  channels: per thread, threads: per workgroup.
template <typename TM>
AddJob<TM> add_job(const Dims &D, const TM *In, int ldi, const Taps &taps, TM *Out, int ldo, int channels, int threads)
{
    const int cblocks = (D.C + 63) / 64, pairs = (D.W + 1) / 2, groups = (pairs + channels - 1) / channels, per = threads / 64;
    const long waves = (long)D.B * ((D.H + kLceRows - 1) / kLceRows) * groups, blocks = (waves + per - 1) / per * cblocks;
    const bool fits = (long)D.W * std::max(ldi, ldo) * (long)sizeof(TM) < (1L << 31) && waves + per < (1L << 31) && blocks < 0x7ffffff0L;
    return AddJob<TM>{In, taps, Out, ldi, ldo, cblocks, fits ? (int)((blocks + 7) / 8 * 8) : 0, groups};
}

// Out += LCE(In), any map; a BRA_* code.
template <typename TM>
int launch_lce(const Dims &D, const TM *In, int ldi, const Taps &taps, TM *Out, int ldo, int kernel_id, hipStream_t st)
{
    const bool two = D.C % 2 == 0;
    const AddJob<TM> J = add_job<TM>(D, In, ldi, taps, Out, ldo, two ? 2 : 1, 256);
    const int cols = two ? 8 : 4;
    const long blocks = ((long)D.B * ((D.H + kLceRows - 1) / kLceRows) * D.W + cols - 1) / cols * J.cblocks;
    if (!J.blocks && blocks > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    const dim3 far((unsigned)((blocks + 7) / 8 * 8)), near((unsigned)J.blocks);
    if (J.blocks && two && J.blocks > 4 * 256 && J.blocks <= 5 * 256) hipLaunchKernelGGL((k_lce<TM, 2, false>), near, dim3(256), 0, st, J, D);
    else if (J.blocks && two) hipLaunchKernelGGL((k_lce<TM, 2, true>), near, dim3(256), 0, st, J, D);
    else if (J.blocks) hipLaunchKernelGGL((k_lce<TM, 1, true>), near, dim3(256), 0, st, J, D);
    else if (two) hipLaunchKernelGGL((k_lce_far<TM, 2>), far, dim3(256), 0, st, In, ldi, taps, Out, ldo, D, J.cblocks);
    else hipLaunchKernelGGL((k_lce_far<TM, 1>), far, dim3(256), 0, st, In, ldi, taps, Out, ldo, D, J.cblocks);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

struct LcePlan {
    int cblocks, height, strips_per_wg, groups;
    long strips;

    __host__ __device__ int blocks() const { return (groups * cblocks + 7) / 8 * 8; }
};

template <typename TM>
struct GradJob {
    const TM *dO, *V;
    Taps taps;
    TM *dV;
    float *Part;
    int ldv, lddv;
    LcePlan p;
};

// About `slots` workgroups of `cols` columns in all, each with the strips of one group.
inline LcePlan lce_plan(const Dims &D, int slots, int cols)
{
    LcePlan p;
    p.cblocks = (D.C + 63) / 64;
    const long want = slots / p.cblocks > 0 ? slots / p.cblocks : 1;
    for (p.height = 20;; p.height /= 2) {            // 20, 10, 5
        p.strips = (long)D.B * ((D.H + p.height - 1) / p.height) * ((D.W + cols - 1) / cols);
        if (p.height == 5 || p.strips >= want) break;
    }
    p.strips_per_wg = (int)((p.strips + want - 1) / want);
    p.groups = (int)((p.strips + p.strips_per_wg - 1) / p.strips_per_wg);
    return p;
}

// ---------------------------------------------------------------------------
// The two gradients of the depth-wise 5x5 correlation (Eq. 7) that read dO with its neighbours:
//     dV[s][c] += sum_{ky,kx} w[c][ky][kx] dO[s - (ky - 2, kx - 2)][c]
//     dWlce[c][ky][kx] = sum_s V[s][c] dO[s - (ky - 2, kx - 2)][c]
// (the second is sum_t dO[t] V[t + (ky - 2, kx - 2)] with s = t + (ky - 2, kx - 2)), so one 5 x 5 window of dO
// serves both and V, dV are touched at the centre only.  Workgroup: 64 channels, 256 VW / 64 neighbouring
// columns; a thread walks down strips of `height` rows of one column with VW channels: a row of 5 values
// enters the window per step, 50 VW FMAs use it, the tap sums stay in registers across the workgroup's strips
// and leave as Part[group][C][25] (k_reduce_parts adds the groups in a fixed order).  Bound by those FMAs
// (and, for VW = 2, by the two wavefronts per SIMD that about 190 registers allow).
// height is a multiple of 5 (the window's rows rotate through fixed registers): 20, or less where that leaves
// too few workgroups (8 x 28 x 28 x 128 float32: 26 us with strips of 20, 128 workgroups).  The next row is requested a step ahead (query
// side with the pass of 60 x 28 x 28 x 96: 99 -> 90 us, 30 x 35 x 35 x 96 87 -> 78).

// Workgroup `block` of J, 256 threads; red: [25][256].  ADDS = false: dV = LCE^T(dO).
template <int VW, bool ADDS, typename TM>
__device__ __forceinline__ void lce_grad_block(const GradJob<TM> &J, const Dims &D, int block, float *red)
{
    constexpr int CPW = 64 / VW, COLS = 256 / CPW;
    const TM *__restrict__ dO = J.dO, *__restrict__ V = J.V;
    TM *__restrict__ dV = J.dV;
    float *__restrict__ Part = J.Part;
    const int ldv = J.ldv, lddv = J.lddv, height = J.p.height, strips_per_wg = J.p.strips_per_wg;
    const long strips = J.p.strips;
    const int cblocks = J.p.cblocks, cb = block % cblocks, c0 = 64 * cb, grp = block / cblocks;
    if (grp * (long)strips_per_wg >= strips) return;
    stage_taps<256>(J.taps, c0, D.C, red);
    const int cl = ((int)threadIdx.x % CPW) * VW, col = threadIdx.x / CPW;
    const bool live = c0 + cl < D.C;
    const int c = live ? c0 + cl : c0;
    float w[25][VW], acc[25][VW];
#pragma unroll
    for (int t = 0; t < 25; ++t)
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            w[t][v] = red[(24 - t) * 64 + (live ? cl : 0) + v];       // window position t meets tap 24 - t
            acc[t][v] = 0.f;
        }
    __syncthreads();
    const int xtiles = (D.W + COLS - 1) / COLS, ytiles = (D.H + height - 1) / height;
    const long first = (long)grp * strips_per_wg, last = min(strips, first + strips_per_wg);
    for (long strip = first; strip < last; ++strip) {
        const int x = (int)(strip % xtiles) * COLS + col, y0 = (int)((strip / xtiles) % ytiles) * height;
        const size_t b = strip / ((long)xtiles * ytiles);
        if (x >= D.W) continue;
        const int y1 = min(y0 + height, D.H);
        const TM *dimg = dO + b * D.N * D.C + c;
        bool xok[5];
        int xc[5];
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
            xok[kx] = (unsigned)(x + kx - 2) < (unsigned)D.W;
            xc[kx] = min(max(x + kx - 2, 0), D.W - 1);
        }
        // rows come from clamped places and are blanked where they are used, not behind the loads
        auto load_row = [&](int y, Channels<VW> (&row)[5]) {
            const size_t first = (size_t)min(max(y, 0), D.H - 1) * D.W;
#pragma unroll
            for (int kx = 0; kx < 5; ++kx) row[kx] = load_channels<VW>(dimg + (first + xc[kx]) * D.C);
        };
        auto blank = [&](int y, const Channels<VW> (&from)[5], Channels<VW> (&row)[5]) {
            const bool in = (unsigned)y < (unsigned)D.H;
#pragma unroll
            for (int kx = 0; kx < 5; ++kx)
#pragma unroll
                for (int v = 0; v < VW; ++v) row[kx].v[v] = in && xok[kx] ? from[kx].v[v] : 0.f;
        };
        Channels<VW> win[5][5], next[5], nv, nd = {};
        auto request = [&](int y) {              // what step y needs
            load_row(y + 2, next);
            const size_t tok = b * D.N + (size_t)min(y, D.H - 1) * D.W + x;
            nv = load_channels<VW>(V + tok * ldv + c);
            if (ADDS) nd = load_channels<VW>(dV + tok * lddv + c);
        };
#pragma unroll
        for (int r = 0; r < 4; ++r) load_row(y0 + r - 2, win[r]);
        request(y0);
#pragma unroll
        for (int r = 0; r < 4; ++r) blank(y0 + r - 2, win[r], win[r]);
        for (int yb = y0; yb < y1; yb += 5) {
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const int y = yb + u;
                if (y >= y1) break;
                blank(y + 2, next, win[(u + 4) % 5]);
                const size_t tok = b * D.N + (size_t)y * D.W + x;
                const Channels<VW> vc = nv;
                Channels<VW> dv = nd;
                request(y + 1);
#pragma unroll
                for (int r = 0; r < 5; ++r)
#pragma unroll
                    for (int kx = 0; kx < 5; ++kx)
#pragma unroll
                        for (int v = 0; v < VW; ++v) {
                            const float d = win[(u + r) % 5][kx].v[v];
                            dv.v[v] = fmaf(w[5 * r + kx][v], d, dv.v[v]);
                            acc[5 * r + kx][v] = fmaf(vc.v[v], d, acc[5 * r + kx][v]);
                        }
                if (live) store_channels<VW>(dV + tok * lddv + c, dv);
            }
        }
    }
    // the columns' sums of a channel through LDS, added in a fixed order: VW rounds of 25 x 256 floats
#pragma unroll
    for (int v = 0; v < VW; ++v) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 25; ++t) red[t * 256 + threadIdx.x] = acc[t][v];
        __syncthreads();
        for (int e = threadIdx.x; e < 25 * CPW; e += 256) {
            const int t = e / CPW, q = e % CPW, ch = c0 + q * VW + v;
            float s = 0.f;
            for (int k = 0; k < COLS; ++k) s += red[t * 256 + k * CPW + q];
            if (ch < D.C) Part[((size_t)grp * D.C + ch) * 25 + 24 - t] = s;
        }
    }
}

template <typename TM, int VW>
__global__ __launch_bounds__(256) void k_lce_grad(GradJob<TM> J, Dims D)
{
    __shared__ float red[25 * 256];
    lce_grad_block<VW, true>(J, D, mfma::swizzled_block(), red);
}

// Launch of k_lce_grad (Part: p.groups arrays of 25 C floats); a BRA_* code.
template <typename TM>
int launch_lce_grad(const Dims &D, const GradJob<TM> &J, hipStream_t st)
{
    const dim3 grid((unsigned)J.p.blocks());
    if (D.C % 2 == 0) hipLaunchKernelGGL((k_lce_grad<TM, 2>), grid, dim3(256), 0, st, J, D);
    else hipLaunchKernelGGL((k_lce_grad<TM, 1>), grid, dim3(256), 0, st, J, D);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// bf16 maps with an even number of channels (bra_lce.hip), on the two-element bf16 dot product: O += LCE(V);
// the passes of the gradients (backward_jobs) leave the tap gradients as lce_grad_groups_bf16 arrays of 25 C floats.
int lce_add_bf16(const Dims &D, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, int ldo, int kernel_id, hipStream_t st);
// LCE(V) in float32, the upper halves of the bits in O and the lower ones in Low, and beside it in the same launch the rows of
// A^r from Q^r, K^r [B, R, C] and their top-k.
int route_rows_lce_bf16(const Dims &D, const float *Qr, const float *Kr, int32_t *Ir, const bf16_t *V, const bf16_t *Wlce, bf16_t *O,
                        bf16_t *Low, hipStream_t st);
int lce_grad_groups_bf16(const Dims &D, int lddv);

}  // namespace lce
}  // namespace bra
