// The depth-wise 5 x 5 correlation (LCE, Eq. 7) and its gradients over whole token maps (internal): threads
// walk down image columns with the window in registers; no halo tiles, no barriers between rows.  The
// kernels of this header take float32 or bf16 maps and any channel count; bra_lce.hip has the bf16 ones for
// even channel counts.
#pragma once

#include "bra_mfma_dev.h"

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

// ---------------------------------------------------------------------------
// Out[t][c] += sum_{ky,kx} w[c][ky][kx] In[t + (ky - 2, kx - 2)][c] over the H x W map (zero outside):
// LCE (Eq. 7).  Workgroup: 64 channels of 256 VW / 64 column pieces; a thread walks down kLceRows rows of one
// column with VW (2 or 1) channels: an input row of 5 columns is read once and goes into the output rows it
// belongs to.  The taps pass through LDS once per workgroup: read per thread from the [C][25] tensor they would
// cost a cache line per lane.  (Requesting all 40 values first, or a row ahead, was no faster: 21 and 23 against 17 us
// on a 16 x 56 x 56 x 64 map; the registers cost more wavefronts than the latency they hide.)
// Row pitches ldi, ldo.
constexpr int kLceRows = 4;

template <typename TM, typename TW, int VW>
__global__ __launch_bounds__(256) void k_lce(const TM *__restrict__ In, int ldi, const TW *__restrict__ Wlce,
                                             TM *__restrict__ Out, int ldo, Dims D, int cblocks)
{
    __shared__ float taps[25][64];
    constexpr int CPW = 64 / VW, COLS = 256 / CPW;
    const int block = mfma::swizzled_block(), cb = block % cblocks, c0 = 64 * cb, yb_n = (D.H + kLceRows - 1) / kLceRows;
    for (int e = threadIdx.x; e < min(64, D.C - c0) * 25; e += 256) taps[e % 25][e / 25] = load_f32(Wlce + (size_t)c0 * 25 + e);
    __syncthreads();
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
        for (int v = 0; v < VW; ++v) w[t][v] = taps[t][cl + v];
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

// Launch of k_lce; a BRA_* code.
template <typename TM, typename TW>
int launch_lce(const Dims &D, const TM *In, int ldi, const TW *Wlce, TM *Out, int ldo, int kernel_id, hipStream_t st)
{
    const int cblocks = (D.C + 63) / 64;
    const long pieces = (long)D.B * ((D.H + kLceRows - 1) / kLceRows) * D.W;
    const bool pairs = D.C % 2 == 0;
    const int cols = pairs ? 8 : 4;
    const long blocks = (pieces + cols - 1) / cols * cblocks;
    if (blocks > 0x7ffffff0L) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    if (pairs) hipLaunchKernelGGL((k_lce<TM, TW, 2>), dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, st, In, ldi, Wlce, Out, ldo, D, cblocks);
    else hipLaunchKernelGGL((k_lce<TM, TW, 1>), dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, st, In, ldi, Wlce, Out, ldo, D, cblocks);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
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
// too few workgroups (8 x 28 x 28 x 128 float32: 26 us with strips of 20, 128 workgroups).

template <typename TM, typename TW, int VW>
__global__ __launch_bounds__(256) void k_lce_grad(const TM *__restrict__ dO, const TM *__restrict__ V, int ldv,
                                                  const TW *__restrict__ Wlce, TM *__restrict__ dV, int lddv,
                                                  float *__restrict__ Part, Dims D, int cblocks, long strips,
                                                  int strips_per_wg, int height)
{
    constexpr int CPW = 64 / VW, COLS = 256 / CPW;
    __shared__ float red[25 * 256];
    const int block = mfma::swizzled_block(), cb = block % cblocks, c0 = 64 * cb, grp = block / cblocks;
    if (grp * (long)strips_per_wg >= strips) return;
    for (int e = threadIdx.x; e < min(64, D.C - c0) * 25; e += 256) red[(e % 25) * 64 + e / 25] = load_f32(Wlce + (size_t)c0 * 25 + e);
    __syncthreads();
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
        Channels<VW> win[5][5];
        auto load_row = [&](int y, Channels<VW> (&row)[5]) {
            const bool in = (unsigned)y < (unsigned)D.H;
#pragma unroll
            for (int kx = 0; kx < 5; ++kx) {
                const int xx = x + kx - 2;
                const bool ok = in && (unsigned)xx < (unsigned)D.W;
                row[kx] = load_channels<VW>(dimg + (size_t)(ok ? y * D.W + xx : 0) * D.C);
#pragma unroll
                for (int v = 0; v < VW; ++v) row[kx].v[v] = ok ? row[kx].v[v] : 0.f;
            }
        };
#pragma unroll
        for (int r = 0; r < 4; ++r) load_row(y0 + r - 2, win[r]);
        for (int yb = y0; yb < y1; yb += 5) {
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const int y = yb + u;
                if (y >= y1) break;
                load_row(y + 2, win[(u + 4) % 5]);
                const size_t tok = b * D.N + (size_t)y * D.W + x;
                const Channels<VW> vc = load_channels<VW>(V + tok * ldv + c);
                Channels<VW> dv = load_channels<VW>(dV + tok * lddv + c);
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

struct LcePlan {
    int cblocks, height, strips_per_wg, groups;
    long strips;
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

// Launch of k_lce_grad (Part: lce_plan(D, slots).groups arrays of 25 C floats); a BRA_* code.
template <typename TM, typename TW>
int launch_lce_grad(const Dims &D, const LcePlan &p, const TM *dO, const TM *V, int ldv, const TW *Wlce, TM *dV, int lddv,
                    float *Part, hipStream_t st)
{
    const dim3 grid((unsigned)((p.groups * p.cblocks + 7) / 8 * 8));
    if (D.C % 2 == 0)
        hipLaunchKernelGGL((k_lce_grad<TM, TW, 2>), grid, dim3(256), 0, st, dO, V, ldv, Wlce, dV, lddv, Part, D, p.cblocks,
                           p.strips, p.strips_per_wg, p.height);
    else
        hipLaunchKernelGGL((k_lce_grad<TM, TW, 1>), grid, dim3(256), 0, st, dO, V, ldv, Wlce, dV, lddv, Part, D, p.cblocks,
                           p.strips, p.strips_per_wg, p.height);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// bf16 maps with an even number of channels (bra_lce.hip), on the two-element bf16 dot product: O += LCE(V);
// the passes of the gradients (backward_jobs) leave the tap gradients as lce_grad_groups_bf16 arrays of 25 C floats.
int lce_add_bf16(const Dims &D, const bf16_t *V, const bf16_t *Wlce, bf16_t *O, int ldo, int kernel_id, hipStream_t st);
// O = LCE(V), and beside it in the same launch the rows of A^r from Q^r, K^r [B, R, C] and their top-k.
int route_rows_lce_bf16(const Dims &D, const float *Qr, const float *Kr, int32_t *Ir, const bf16_t *V, const bf16_t *Wlce, bf16_t *O,
                        hipStream_t st);
int lce_grad_groups_bf16(const Dims &D, int lddv);

}  // namespace lce
}  // namespace bra
