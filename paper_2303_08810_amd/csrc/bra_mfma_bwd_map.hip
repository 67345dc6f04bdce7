// Attention backward for maps small enough that one head's Q, K, V and dO of a whole image fit in LDS (bf16, heads of
// 32 channels, regions of at most 16 tokens, e.g. the third and fourth stages of the paper's backbones).
//
// Small regions route to many others: a workgroup per region (k_attn_bwd_q, k_attn_bwd_kv) copies every K, V row of the
// image about k times and every Q, dO row as often again, 308 + 308 MB from the L2s for a 64 x 14 x 14 x 384 map with
// k = 16 (60 + 100 us).  Here workgroup (image, head) copies the four slices once, its wavefronts walk over the query
// regions (O, dQ and the row statistics, which stay in LDS) and then over the key regions (dK, dV), all rows found by
// index in LDS.  Arithmetic, operand layouts and rounding are those of the per-region kernels.
// 67 us at that shape.  Bound by LDS reads: every row is read as an operand row and by the transposing read on each side.
// The depth-wise parts come from the same slices at its end, in registers while other wavefronts still have key regions; they were a launch that read V, dO, O and
// dV again.  Whole gradient (us) with that launch / now: 64 x 14 x 14 x 384, k = 16 168.4 / 167.3 (on another machine 158.8 / 156.2), 64 x 14 x 14 x 256 109.4 / 106.2,
// 128 x 14 x 14 x 64 63.3 / 57.3, 32 x 14 x 28 x 256 105.6 / 99.8, 128 x 7 x 7 x 256, k = 9 109.8 / 102.8, 512 x 7 x 7 x 64 101.2 / 94.3.  At its head instead, parked in the places of O and
// dV in 2-byte stores: 161 / 169 at the first shape; one after the other behind the barrier 166.
// (Scores on 4x4x4 products, so that none of the 16 tile columns idles at 4 tokens per region, read the same bytes:
// 67 us at 128 registers, 84 at 144.)
#include "bra_bwd_dev.h"
#include "bra_lce_region.h"
#include "bra_mfma_bwd_map.h"

namespace bra {

using namespace mfma;

namespace {

constexpr int kPitch = 40;       // 32 channels + 8: rows of 80 bytes
constexpr int kWaveBytes = 768;  // of a wavefront's own: rows of a block, lse and D of its queries
constexpr int kParkPitch = 36;   // floats per token of the depth-wise sums
constexpr size_t kTapBytes = 25 * 32 * 4;   // tap gradients of a wavefront

struct MapSmem {
    size_t rows, first, list, start, count, lse, dsum, wave, zero, bytes;
};

__host__ __device__ inline MapSmem map_smem(int N, int R, int k, int waves, bool conv)
{
    MapSmem m;
    size_t off = (size_t)4 * N * kPitch * 2;
    auto take = [&](size_t bytes) { const size_t at = off; off += (bytes + 15) & ~(size_t)15; return at; };
    m.rows = take((size_t)R * k * 4);
    m.first = take((size_t)R * 4);
    m.list = take((size_t)2 * R * k * 4);
    m.start = take((size_t)(R + 1) * 4);
    m.count = take((size_t)R * 4);
    m.lse = take((size_t)N * 4);
    m.dsum = take((size_t)N * 4);
    m.wave = take((size_t)waves * kWaveBytes);
    m.zero = take(16);
    m.bytes = conv && off < waves * kTapBytes ? waves * kTapBytes : off;
    return m;
}

// acc[dt] += T^T[channel 16 dt + 4 g + j][..] x vals for 64 gathered rows of T: row[tp][half] starts the row of this
// lane's transposing read (contraction slots as in the accumulator layout of vals).
__device__ __forceinline__ void rows_contract(const bf16_t *T, const int (&row)[2][2], const float (&vals)[4][4], int i,
                                              f32x4 (&acc)[2])
{
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
        const float pv[8] = {vals[2 * tp][0], vals[2 * tp][1], vals[2 * tp][2], vals[2 * tp][3],
                             vals[2 * tp + 1][0], vals[2 * tp + 1][1], vals[2 * tp + 1][2], vals[2 * tp + 1][3]};
        const bf16x8 pb = pack8(pv);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const int col = 16 * dt + 4 * (i % 4);
            const u32x2 a0 = __builtin_bit_cast(u32x2, lds_read_tr16(T + row[tp][0] + col));
            const u32x2 a1 = __builtin_bit_cast(u32x2, lds_read_tr16(T + row[tp][1] + col));
            acc[dt] = mfma16(__builtin_bit_cast(bf16x8, u32x4{a0[0], a0[1], a1[0], a1[1]}), pb, acc[dt]);
        }
    }
}

// What a workgroup works on, staged in LDS.
struct MapWork {
    int h, b;
    bf16_t *Qs, *Ks, *Vs, *Gs;       // [N][kPitch]: the head's slices of Q, K, V, dO
    int *rows;                       // [R][k]: first token of the routed regions
    int *first;                      // [R]: first token of a region
    int *start, *named;              // key region j is named by query regions named[start[j] .. start[j + 1])
    float *lse, *dsum;               // [N]: row statistics
    char *wave_mem;
    bf16_t *zero;                    // 16 bytes of zeros
};

template <int NW>
__device__ __forceinline__ bool map_stage(MapWork &w, char *smem, const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                          const bf16_t *__restrict__ V, const bf16_t *__restrict__ dO,
                                          const int32_t *__restrict__ Ir, const Dims &D, int total)
{
    constexpr int T = 64 * NW;
    const int wid = swizzled_block();            // the heads of an image share the memory lines of its rows
    if (wid >= total) return false;
    w.h = wid % D.heads;
    w.b = wid / D.heads;
    const int C = D.C, entries = D.R * D.k;
    const MapSmem L = map_smem(D.N, D.R, D.k, NW, false);
    w.Qs = (bf16_t *)smem;
    w.Ks = w.Qs + (size_t)D.N * kPitch;
    w.Vs = w.Ks + (size_t)D.N * kPitch;
    w.Gs = w.Vs + (size_t)D.N * kPitch;
    w.rows = (int *)(smem + L.rows);
    w.first = (int *)(smem + L.first);
    w.start = (int *)(smem + L.start);
    int *list = (int *)(smem + L.list), *count = (int *)(smem + L.count), *arrived = list + entries;
    w.named = arrived;
    w.lse = (float *)(smem + L.lse);
    w.dsum = (float *)(smem + L.dsum);
    const int tid = threadIdx.x;
    w.wave_mem = smem + L.wave + (tid / kWave) * kWaveBytes;
    w.zero = (bf16_t *)(smem + L.zero);
    if (tid < 8) w.zero[tid] = 0;
    const size_t img = (size_t)w.b * D.N * C + 32 * w.h;
    const float s_inv = 1.0f / (float)D.S;
    // f(entry, region it names) for this thread's routing entries; the first ones are requested ahead of the slices
    const int32_t *irb = Ir + (size_t)w.b * entries;
    int named[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) named[u] = irb[min(tid + T * u, entries - 1)];
    auto each_entry = [&](auto f) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (tid + T * u < entries) f(tid + T * u, region_index(named[u], D.R));
        for (int e = tid + 2 * T; e < entries; e += T) f(e, region_index(irb[e], D.R));
    };
    // the head's slices of the four maps
    const int chunks = D.N * 4;
    for (int c0 = 0; c0 < chunks; c0 += 2 * T) {
        u32x4 r[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int idx = min(c0 + tid + T * u, chunks - 1);
            const size_t at = img + (size_t)(idx / 4) * C + (idx % 4) * 8;
            r[u][0] = *(const u32x4 *)(Q + at);
            r[u][1] = *(const u32x4 *)(K + at);
            r[u][2] = *(const u32x4 *)(V + at);
            r[u][3] = *(const u32x4 *)(dO + at);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int idx = c0 + tid + T * u;
            if (idx < chunks) {
                bf16_t *dst = w.Qs + (idx / 4) * kPitch + (idx % 4) * 8;
#pragma unroll
                for (int m = 0; m < 4; ++m) *(u32x4 *)(dst + (size_t)m * D.N * kPitch) = r[u][m];
            }
        }
    }
    for (int r = tid; r < D.R; r += T) {
        const int ry = fast_div(r, s_inv);
        w.first[r] = ry * D.rh * D.W + (r - ry * D.S) * D.rw;
        count[r] = 0;
    }
    __syncthreads();
    // routing rows as token numbers, and per key region the query regions that name it, in the order of the entries:
    // arrival order through a counter, then a rank among the (few) entries of the same region
    each_entry([&](int e, int j) {
        w.rows[e] = w.first[j];
        arrived[e] = atomicAdd(&count[j], 1);
    });
    __syncthreads();
    for (int j = tid; j <= D.R; j += T) {
        int s = 0;
#pragma unroll 8
        for (int u = 0; u < j; ++u) s += count[u];
        w.start[j] = s;
    }
    __syncthreads();
    each_entry([&](int e, int j) { list[w.start[j] + arrived[e]] = e; });
    __syncthreads();
    each_entry([&](int e, int j) {
        const int s0 = w.start[j], s1 = w.start[j + 1];
        int rank = 0;
#pragma unroll 8
        for (int u = s0; u < s1; ++u) rank += list[u] < e;
        arrived[s0 + rank] = e / D.k;            // `arrived` becomes the ordered list of query regions
    });
    return true;      // the key side reads the list behind the next barrier
}

// CONV: with the depth-wise parts.  Four wavefronts per SIMD, two workgroups of 8 to a compute unit, spill 6 registers; a bound of two spills none and takes the same time with CONV
// (128 registers; 64 x 14 x 14 x 384 148.2 us, 148.3), without it 134 registers leave one workgroup (1024 x 14 x 14 x 64 243 -> 285).
template <int NW, bool CONV>
__global__ __launch_bounds__(64 * NW, 4) void k_attn_bwd_map(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                          const bf16_t *__restrict__ V, const bf16_t *__restrict__ dO,
                                                          const int32_t *__restrict__ Ir, bf16_t *__restrict__ O,
                                                          bf16_t *__restrict__ dQKV, const bf16_t *__restrict__ Wlce,
                                                          float *__restrict__ PartLce, Dims D, int total)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    MapWork w;
    if (!map_stage<NW>(w, smem, Q, K, V, dO, Ir, D, total)) return;
    const int h = w.h, b = w.b, C = D.C, n = D.n, kn = D.kn;
    const bf16_t *Qs = w.Qs, *Ks = w.Ks, *Vs = w.Vs, *Gs = w.Gs;
    const int *rows = w.rows, *first = w.first, *start = w.start, *arrived = w.named;
    float *lse_s = w.lse, *dsum_s = w.dsum;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, g = lane / 16, i = lane % 16;
    int *tokw = (int *)w.wave_mem;
    float *wl = (float *)(tokw + 64), *wd = wl + 64;
    const size_t img = (size_t)b * D.N * C + 32 * h;
    const float rw_inv = 1.0f / (float)D.rw, n_inv = 1.0f / (float)n;
    auto in_region = [&](int slot) {             // token offset of a slot from its region's first token
        const int sy = fast_div(slot, rw_inv);
        return sy * D.W + slot - sy * D.rw;
    };
    const float c_exp = D.scale * 1.4426950408889634f;
    const int nblocks = (kn + 63) / 64;
    const int my_q = in_region(min(i, n - 1));
    // ---- query regions: O, dQ, row statistics
    for (int reg = wave; reg < D.R; reg += NW) {
        const int tok = first[reg] + my_q;
        const bf16x8 qf = *(const bf16x8 *)(Qs + tok * kPitch + 8 * g), gf = *(const bf16x8 *)(Gs + tok * kPitch + 8 * g);
        float m = -INFINITY, l = 0.f, dd = 0.f;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        for (int step = 0; step < 2 * nblocks; ++step) {
            const int sweep = step >= nblocks ? 1 : 0, k0 = 64 * (step - sweep * nblocks);
            if (step == 0 || nblocks > 1) {
                const int key = min(k0 + lane, kn - 1), p = fast_div(key, n_inv);
                tokw[lane] = (rows[reg * D.k + p] + in_region(key - p * n)) * kPitch;
            }
            int row[2][2];
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int half = 0; half < 2; ++half) row[tp][half] = tokw[32 * tp + 16 * half + 4 * g + i / 4];
            f32x4 s[4], dp[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int kr = tokw[16 * t + i];
                const bf16x8 kf = *(const bf16x8 *)(Ks + kr + 8 * g), vf = *(const bf16x8 *)(Vs + kr + 8 * g);
                s[t] = mfma16(kf, qf, f32x4{0.f, 0.f, 0.f, 0.f});      // S^T[key 16 t + 4 g + j][query i]
                dp[t] = mfma16(vf, gf, f32x4{0.f, 0.f, 0.f, 0.f});     // dP^T
            }
            const int left = kn - k0;
            if (left < 64) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[t][j] = 16 * t + 4 * g + j >= left ? -INFINITY : s[t][j];
            }
            float e[4][4];
            if (sweep == 0) {
                float mx = s[0][0];
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) mx = fmaxf(mx, s[t][j]);
                const float m_new = fmaxf(m, cross_row_max(mx));          // finite: the block's first key exists
                const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c_exp);
                m = m_new;
                const float mc = m * c_exp;
                float ls = 0.f, ds = 0.f;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        e[t][j] = __builtin_amdgcn_exp2f(fmaf(s[t][j], c_exp, -mc));
                        ls += e[t][j];
                        ds = fmaf(e[t][j], dp[t][j], ds);
                    }
                l = fmaf(l, alpha, cross_row_sum(ls));
                dd = fmaf(dd, alpha, cross_row_sum(ds));
                if (step) {
                    acc[0] *= alpha;
                    acc[1] *= alpha;
                }
                rows_contract(Vs, row, e, i, acc);
                if (step + 1 < nblocks) continue;
                const float inv = 1.0f / l;
                dd *= inv;
                if (i < n) {
                    bf16_t *orow = O + img + (size_t)tok * C + 4 * g;
                    *(u32x2 *)orow = pack4(acc[0] * inv);
                    *(u32x2 *)(orow + 16) = pack4(acc[1] * inv);
                    if (g == 0) {
                        lse_s[tok] = mc + __builtin_amdgcn_logf(l);       // v_log_f32: log2
                        dsum_s[tok] = dd;
                    }
                }
                acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (nblocks > 1) continue;
            } else {
                const float mc = m * c_exp;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) e[t][j] = __builtin_amdgcn_exp2f(fmaf(s[t][j], c_exp, -mc));
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) e[t][j] *= dp[t][j] - dd;
            rows_contract(Ks, row, e, i, acc);           // times scale / l at the end
            if (nblocks == 1) break;
        }
        if (i < n) {
            const float f = D.scale / l;
            bf16_t *qrow = dQKV + ((size_t)b * D.N + tok) * 3 * C + 32 * h + 4 * g;
            *(u32x2 *)qrow = pack4(acc[0] * f);
            *(u32x2 *)(qrow + 16) = pack4(acc[1] * f);
        }
    }
    __syncthreads();
    // ---- key regions: dK, dV
    for (int reg = wave; reg < D.R; reg += NW) {
        const int tok = first[reg] + my_q;
        const bf16x8 kf = *(const bf16x8 *)(Ks + tok * kPitch + 8 * g), vf = *(const bf16x8 *)(Vs + tok * kPitch + 8 * g);
        const int l0 = start[reg], nrows = (start[reg + 1] - l0) * n;
        f32x4 ak[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, av[2] = {ak[0], ak[0]};
        for (int r0 = 0; r0 < nrows; r0 += 64) {
            {
                const int r = min(r0 + lane, nrows - 1), p = fast_div(r, n_inv);
                const int qt = first[arrived[l0 + p]] + in_region(r - p * n);
                tokw[lane] = qt * kPitch;
                wl[lane] = r0 + lane < nrows ? lse_s[qt] : INFINITY;       // a missing row: P = exp2(-inf) = 0
                wd[lane] = dsum_s[qt];
            }
            int row[2][2];
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int half = 0; half < 2; ++half) row[tp][half] = tokw[32 * tp + 16 * half + 4 * g + i / 4];
            float p[4][4], ds[4][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int qr = tokw[16 * t + i];
                const bf16x8 qf = *(const bf16x8 *)(Qs + qr + 8 * g), gf = *(const bf16x8 *)(Gs + qr + 8 * g);
                const f32x4 s = mfma16(qf, kf, f32x4{0.f, 0.f, 0.f, 0.f});       // S[query 16 t + 4 g + j][key i]
                const f32x4 dp = mfma16(gf, vf, f32x4{0.f, 0.f, 0.f, 0.f});
                const f32x4 l4 = *(const f32x4 *)(wl + 16 * t + 4 * g), d4 = *(const f32x4 *)(wd + 16 * t + 4 * g);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    p[t][j] = __builtin_amdgcn_exp2f(fmaf(s[j], c_exp, -l4[j]));
                    ds[t][j] = p[t][j] * (dp[j] - d4[j]);
                }
            }
            rows_contract(Gs, row, p, i, av);
            rows_contract(Qs, row, ds, i, ak);
        }
        if (i < n) {
            bf16_t *krow = dQKV + ((size_t)b * D.N + tok) * 3 * C + C + 32 * h + 4 * g;
            *(u32x2 *)krow = pack4(ak[0] * D.scale);
            *(u32x2 *)(krow + 16) = pack4(ak[1] * D.scale);
            *(u32x2 *)(krow + C) = pack4(av[0]);
            *(u32x2 *)(krow + C + 16) = pack4(av[1]);
        }
    }
    if (!CONV) return;
    // ---- the depth-wise parts of the head's channels, from the slices (SliceItem; a wavefront has one pair of items at most), in registers while
    // others still have key regions
    const int quads = (D.W + 3) / 4, items = quads * ((D.H + 3) / 4), pairs = (items + 1) / 2;
    const int first_taps = 2 * pairs <= NW ? pairs : 0;      // with wavefronts to spare, others take the tap gradients
    const float q_inv = 1.0f / (float)quads;
    float o[2][4][4], acc[25];
    if (wave < pairs) {
        const lce::SliceItem item(D, 2 * wave, items, quads, q_inv, lane, kPitch);
        const lce::LaneTaps<false> forward(Wlce, 32 * h + lane % 32);
        const lce::LaneTaps<true> reversed(Wlce, 32 * h + lane % 32);
        unsigned wt[5][3];
        forward.operands(wt);
        item.sums(Vs, w.zero, D, kPitch, wt, o[0]);
        reversed.operands(wt);
        item.sums(Gs, w.zero, D, kPitch, wt, o[1]);
    }
    const bool has_taps = wave >= first_taps && wave - first_taps < pairs;
    if (has_taps) {
#pragma unroll
        for (int t = 0; t < 25; ++t) acc[t] = 0.f;
        lce::SliceItem(D, 2 * (wave - first_taps), items, quads, q_inv, lane, kPitch).taps(Gs, Vs, w.zero, D, kPitch, acc);
    }
    __syncthreads();                             // the slices have been read; O and dV are there
    float *parked = (float *)smem;               // [2][N][kParkPitch], where the slices were
    constexpr int CHUNKS = 2;
    u32x4 *to[CHUNKS][2], add[CHUNKS][2];
    auto places = [&](int e, u32x4 *(&at)[2]) {
        at[0] = (u32x4 *)(O + img + (size_t)(e / 4) * C + e % 4 * 8);
        at[1] = (u32x4 *)(dQKV + ((size_t)b * D.N + e / 4) * 3 * C + 2 * C + 32 * h + e % 4 * 8);
    };
    const int chunks = 4 * D.N;
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
        places(min((int)threadIdx.x + 64 * NW * u, chunks - 1), to[u]);
        add[u][0] = *to[u][0];
        add[u][1] = *to[u][1];
    }
    if (wave < pairs) {
        const lce::SliceItem item(D, 2 * wave, items, quads, q_inv, lane, kPitch);
        float *at = parked + (item.y0 * D.W + item.x0) * kParkPitch + lane % 32;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (item.mine && item.y0 + a < D.H && item.x0 + c < D.W) {
                    at[(a * D.W + c) * kParkPitch] = o[0][a][c];
                    at[(D.N + a * D.W + c) * kParkPitch] = o[1][a][c];
                }
    }
    __syncthreads();
    auto sum = [&](int e, int which, u32x4 v) {
        const f32x4 *f = (const f32x4 *)(parked + (which * D.N + e / 4) * kParkPitch + e % 4 * 8);
        const f32x4 lo = f[0], hi = f[1];
        const float r[8] = {bf16_lo(v[0]) + lo[0], bf16_hi(v[0]) + lo[1], bf16_lo(v[1]) + lo[2], bf16_hi(v[1]) + lo[3],
                            bf16_lo(v[2]) + hi[0], bf16_hi(v[2]) + hi[1], bf16_lo(v[3]) + hi[2], bf16_hi(v[3]) + hi[3]};
        return __builtin_bit_cast(u32x4, pack8(r));
    };
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
        const int e = threadIdx.x + 64 * NW * u;
        if (e >= chunks) break;
        *to[u][0] = sum(e, 0, add[u][0]);
        *to[u][1] = sum(e, 1, add[u][1]);
    }
    for (int e = threadIdx.x + 64 * NW * CHUNKS; e < chunks; e += 64 * NW) {
        u32x4 *at[2];
        places(e, at);
        *at[0] = sum(e, 0, *at[0]);
        *at[1] = sum(e, 1, *at[1]);
    }
    // ---- the image's sums of the tap gradients
    float *sums = (float *)smem;                 // [pair of items][tap][channel]
    __syncthreads();
    if (has_taps) {
#pragma unroll
        for (int t = 0; t < 25; ++t) {
            const float v = acc[t] + __shfl_xor(acc[t], 32);
            if (lane < 32) sums[((wave - first_taps) * 25 + t) * 32 + lane] = v;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 25 * 32; e += 64 * NW) {
        const int c = e / 25, t = e - 25 * c;
        float s = 0.f;
        for (int u = 0; u < pairs; ++u) s += sums[(u * 25 + 24 - t) * 32 + c];
        PartLce[((size_t)b * C + 32 * h) * 25 + e] = s;
    }
}

int waves_of(const Dims &D)
{
    // 16 wavefronts where only one workgroup fits a compute unit's LDS or there is at most one per unit; else two of 8
    return map_smem(D.N, D.R, D.k, 8, false).bytes > (size_t)kMaxLds / 2 || (long)D.B * D.heads <= 256 ? 16 : 8;
}

template <int NW, bool CONV>
int launch(const Dims &D, const bf16_t *Q, const bf16_t *K, const bf16_t *V, const bf16_t *dO, const int32_t *Ir, bf16_t *O,
           bf16_t *dQKV, const bf16_t *Wlce, float *PartLce, hipStream_t st)
{
    static bool opted = false;
    if (!opted) {
        if (hipFuncSetAttribute((const void *)k_attn_bwd_map<NW, CONV>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess)
            return BRA_ERR_LAUNCH;
        opted = true;
    }
    const int total = D.B * D.heads;
    hipLaunchKernelGGL((k_attn_bwd_map<NW, CONV>), dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * NW), map_smem(D.N, D.R, D.k, NW, CONV).bytes,
                       st, Q, K, V, dO, Ir, O, dQKV, Wlce, PartLce, D, total);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace

bool attn_bwd_map_ok(const Dims &D)
{
    // regions of up to 8 tokens: larger ones fill the per-region kernels' tiles and gather each row fewer times
    // and few workgroups leave the chip idle: by images / by regions, whole gradient (us), 128 of them: 64 x 7 x 7 x 64, k = 16
    // 42.0 / 37.1; 64 x 14 x 14 x 64, k = 44 88 / 78; 64 x 14 x 28 x 64, k = 16 80 / 73; 192: 24 x 14 x 14 x 256, k = 16 71.6 /
    // 76.9; 8 x 7 x 7 x 768, k = 44 70.8 / 81.2
    return D.d == 32 && (long)D.B * D.heads >= 160 && D.n <= 8 && D.k > 1 && (long)D.B * D.heads < 0x7ffffff0L && map_smem(D.N, D.R, D.k, 16, false).bytes <= (size_t)kMaxLds;
}

// Wherever each pair of items has a wavefront, on sides that the items' tap gradients take, while there are few rounds of workgroups: in many, the
// wavefronts without a pair hold their places until the others are done, and the tap gradients of every image are an array to be summed.  Whole gradient (us), here / with the
// launch, by (image, head) pairs: 4 x 4 x 64 (1 pair of items) 1024 54 / 55, 1536 70 / 68, 4096 151 / 137; 7 x 7 x 64 (2) 1024 91 / 98, 4096 295 / 296, 8192 591 / 569; 7 x 14 x 64 (4) 1024
// 106 / 109, 2048 189 / 184; 14 x 14 x 64 (8) 768 107 / 109, 1024 133 / 131, 2048 257 / 239; 16 x 16 x 512 (8) 512 145 / 150, 768 212 / 212, 1024 281 / 276; 14 x 28 x 256 (14), where a
// compute unit holds one workgroup, 192 78 / 82, 320 124 / 120, 1024 312 / 298.
bool attn_bwd_map_convolves(const Dims &D)
{
    const int items = (D.W + 3) / 4 * ((D.H + 3) / 4), waves = waves_of(D);
    const long most = waves == 16 ? 256 : items > 8 ? 768 : items > 2 && items <= 4 && D.N > 32 ? 4096 : 1024;
    return D.H >= 4 && D.W >= 4 && items <= 2 * waves && (long)D.B * D.heads <= most;
}

int launch_attn_bwd_map(const Dims &D, const bf16_t *Q, const bf16_t *K, const bf16_t *V, const bf16_t *dO, const int32_t *Ir,
                        bf16_t *O, bf16_t *dQKV, const bf16_t *Wlce, float *PartLce, int kernel_id, hipStream_t st)
{
    ProfScope ps(st, kernel_id);
    const bool conv = attn_bwd_map_convolves(D);
    const auto run = waves_of(D) == 16 ? (conv ? launch<16, true> : launch<16, false>) : conv ? launch<8, true> : launch<8, false>;
    return run(D, Q, K, V, dO, Ir, O, dQKV, Wlce, PartLce, st);
}

}  // namespace bra
