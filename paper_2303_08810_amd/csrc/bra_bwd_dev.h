// Device-side pieces of the backward pass that both kernel families use (internal): the depth-wise
// correlation's gradients for float32 and bf16 maps, the list of query regions that attend to a key region,
// and the reduction of per-workgroup partial sums.
#pragma once

#include "bra_mfma_dev.h"

namespace bra {
namespace bwd {

using mfma::bf16_hi;
using mfma::bf16_lo;
using mfma::f32x2;
using mfma::kWave;

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
    const int cb = blockIdx.x % cblocks, c0 = 64 * cb, grp = blockIdx.x / cblocks;
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

// About `slots` workgroups in all, each with the strips of one group.
inline LcePlan lce_plan(const Dims &D, int slots)
{
    const int cols = D.C % 2 == 0 ? 8 : 4;
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
// The entries of rows `irb` (D.R x D.k of one image) with value j among entries [e0, e0 + kListChunk), in
// ascending order, to `list`; returns how many.  Called by all 256 threads; ends with a barrier.  The order is
// that of the entry numbers, so sums over the list come out the same every time.
constexpr int kListChunk = 1024;

__device__ __forceinline__ int collect_entries(const int32_t *__restrict__ irb, int entries, int e0, int j, int R,
                                               int *list, int *counts)
{
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    unsigned long long votes[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = e0 + 256 * u + (int)threadIdx.x;
        votes[u] = __ballot(e < entries && region_index(irb[e < entries ? e : 0], R) == j);
        if (lane == 0) counts[4 * u + wave] = __popcll(votes[u]);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == wave && (votes[u] >> lane & 1))
                list[total + __popcll(votes[u] & ((1ull << lane) - 1))] = e0 + 256 * u + (int)threadIdx.x;
            total += counts[4 * u + w];
        }
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------------------
// out[e] = sum_p part[p][e], p in a fixed order, for up to three arrays in one launch.  A workgroup
// of 1024 threads takes 1024 / slices elements x `slices` slices of p (a power of two up to 32, about
// the number of partial arrays), the slices summed through LDS.
struct ReduceJob {
    const float *part;
    float *out;
    int nparts, count, slices, blocks;
};

inline ReduceJob reduce_job(const float *part, float *out, int nparts, int count)
{
    int slices = 1;
    while (slices < 32 && slices < nparts) slices *= 2;
    const int elems = 1024 / slices;
    return ReduceJob{part, out, nparts, count, slices, (count + elems - 1) / elems};
}

static __global__ __launch_bounds__(1024) void k_reduce_parts(ReduceJob j0, ReduceJob j1, ReduceJob j2)
{
    __shared__ float red[1024];
    int bi = blockIdx.x;
    ReduceJob job = j0;
    if (bi >= j0.blocks) {
        bi -= j0.blocks;
        job = j1;
        if (bi >= j1.blocks) {
            bi -= j1.blocks;
            job = j2;
        }
    }
    const int elems = 1024 / job.slices;
    const int x = threadIdx.x % elems, y = threadIdx.x / elems, e = bi * elems + x;
    float sum = 0.f;
    if (e < job.count)
#pragma unroll 8
        for (int p = y; p < job.nparts; p += job.slices) sum += job.part[(size_t)p * job.count + e];
    red[y * elems + x] = sum;
    __syncthreads();
    if (y == 0 && e < job.count) {
        float total = 0.f;
        for (int u = 0; u < job.slices; ++u) total += red[u * elems + x];
        job.out[e] = total;
    }
}

}  // namespace bwd
}  // namespace bra
