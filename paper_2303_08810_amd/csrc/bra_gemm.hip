// bf16 products of the general pipelines.
#include "bra_attn_dev.h"
#include "bra_gemm.h"
#include "bra_proj_dev.h"

#include <algorithm>
#include <cmath>

namespace bra {

using namespace mfma;

namespace {

// The wait between the last 32x32x16 products and the first use of their results, spelled out: where a branch lies between
// them the compiler has left it short.
__device__ __forceinline__ void products_done()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15");
    __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------
// Out[m][o] = sum_k In[m][k] W[k][o] (W row-major with ldw columns, as the caller holds it), float32 In and Out,
// for a tile of 64 rows m x 32 CW outputs o (128 or 64), the contraction in chunks of 64
// staged in LDS (the next chunk is requested while the current one is multiplied).
// The four wavefronts split the tile 2 x 2 (32 rows x 16 CW outputs each); the product is formed
// transposed on 32x32x16 products (16x16x32 ones, at 27 clocks for half the work of 32, took 5 us more of 8 x 32 x 32 x 768's
// projection launch), with W's columns taken as in k_gemm_dma, so that a lane stores 8 consecutive outputs of one row;
// its W operand (rows = outputs) comes out of the row-major chunk by the transposing LDS read.
// Output column o goes to buffer o / cols (buffers of `cols` columns each, e.g. Q^r, K^r), column o % cols.
// In enters as three exact bf16 terms (smallest first).
constexpr int kGemmPitch = 80;      // bf16 per LDS row of In: 64 + 16 (rows of 160 bytes); W: the tile's width + 16
constexpr int kGemmGroupW = 64;     // W: 128 bytes more after every 8 rows: the neighbouring lane group of a
                                    // transposing read (8 rows further on) then meets the other half of the banks

// Ws: [64 k][32 CW + 16] and 8 group paddings, Xs[q]: [64][P].
constexpr size_t kGemm64Bytes = (size_t)(3 * 64 * kGemmPitch + 64 * (64 + 16) + 8 * kGemmGroupW) * 2;     // CW = 2

template <int CW>
__device__ __forceinline__ void gemm64(const GemmRegions &J, const bf16_t *__restrict__ W, int ldw, int K, int block,
                                       bf16_t *Ws, bf16_t *const (&Xs)[3])
{
    const int M = (int)J.M, Nout = J.Nout;
    constexpr int P = kGemmPitch, NT = 3, COLS = 32 * CW, PW = COLS + 16;
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int otiles = (Nout + COLS - 1) / COLS;
    const int m0 = (block / otiles) * 64, o0 = (block % otiles) * COLS;

    // this thread's pieces of a chunk: 4 x 16 bytes of W and 2 x 8 floats of In
    u32x4 wreg[CW], xreg[4];
    auto request = [&](int k0) {
#pragma unroll
        for (int u = 0; u < CW; ++u) {
            const int idx = tid + 256 * u;                       // (row k, 8 outputs)
            const int o = min(o0 + (idx % (COLS / 8)) * 8, Nout - 8);    // columns past the end repeat the last; never stored
            wreg[u] = *(const u32x4 *)(W + (size_t)(k0 + idx / (COLS / 8)) * ldw + o);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int idx = tid + 256 * u;
            const float *src = J.In + (size_t)min(m0 + idx / 8, M - 1) * K + k0 + (idx % 8) * 8;
            xreg[2 * u] = *(const u32x4 *)src;
            xreg[2 * u + 1] = *(const u32x4 *)(src + 4);
        }
    };
    auto park = [&]() {
#pragma unroll
        for (int u = 0; u < CW; ++u) {
            const int idx = tid + 256 * u;
            const int row = idx / (COLS / 8);
            *(u32x4 *)(Ws + row * PW + (row / 8) * kGemmGroupW + (idx % (COLS / 8)) * 8) = wreg[u];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int idx = tid + 256 * u;
            const int at = (idx / 8) * P + (idx % 8) * 8;
            const f32x4 lo = __builtin_bit_cast(f32x4, xreg[2 * u]), hi = __builtin_bit_cast(f32x4, xreg[2 * u + 1]);
            const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            bf16x8 t[3];
            split3(x, t);
#pragma unroll
            for (int q = 0; q < 3; ++q) *(bf16x8 *)(Xs[q] + at) = t[q];
        }
    };

    // wavefront (wr, wc) owns rows 32 wr .. 32 wr + 31 and outputs 16 CW wc .. + 16 CW - 1 of the workgroup's tile
    const int wr = wave / 2, wc = wave % 2, h = lane / 32, c = lane % 32;
    const int s = lane % 16, q = lane / 16, col4 = (s % 2) * 2 + s % 4 / 2;       // see k_gemm_dma
    f32x16 acc[CW / 2];
#pragma unroll
    for (int t = 0; t < CW / 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    request(0);
    for (int k0 = 0; k0 < K; k0 += 64) {
        if (k0) __syncthreads();          // the previous chunk has been read
        park();
        __syncthreads();
        if (k0 + 64 < K) request(k0 + 64);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 xb[NT];
#pragma unroll
            for (int u = 0; u < NT; ++u) xb[u] = *(const bf16x8 *)(Xs[u] + (32 * wr + c) * P + 16 * ks + 8 * h);
#pragma unroll
            for (int t = 0; t < CW / 2; ++t) {
                u32x2 r[2];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int k = 16 * ks + 8 * (q / 2) + 4 * half + s / 4;
                    r[half] = __builtin_bit_cast(u32x2, lds_read_tr16(Ws + k * PW + (k / 8) * kGemmGroupW + 16 * CW * wc + 32 * t + 16 * (q % 2) + 4 * col4));
                }
                const bf16x8 wf = __builtin_bit_cast(bf16x8, u32x4{r[0][0], r[0][1], r[1][0], r[1][1]});
#pragma unroll
                for (int u = NT - 1; u >= 0; --u) acc[t] = mfma32(wf, xb[u], acc[t]);
            }
        }
    }
    products_done();
    const int m = m0 + 32 * wr + c;
    if (m >= M) return;
#pragma unroll
    for (int t = 0; t < CW / 2; ++t)
#pragma unroll
        for (int run = 0; run < 2; ++run) {
            const int o = o0 + 16 * CW * wc + 32 * t + 16 * run + 8 * h;
            if (o >= Nout) continue;
            const int which = o / J.cols, col = o % J.cols;
            float *dst = J.buf[which] + (size_t)m * J.cols + col;
            *(f32x4 *)dst = f32x4{acc[t][8 * run], acc[t][8 * run + 1], acc[t][8 * run + 2], acc[t][8 * run + 3]};
            *(f32x4 *)(dst + 4) = f32x4{acc[t][8 * run + 4], acc[t][8 * run + 5], acc[t][8 * run + 6], acc[t][8 * run + 7]};
        }
}

// The region-level product on its own.
template <int CW>
__global__ __launch_bounds__(256) void k_gemm(GemmRegions J, const bf16_t *__restrict__ W, int ldw, int K)
{
    __shared__ __attribute__((aligned(16))) bf16_t Ws[64 * (32 * CW + 16) + 8 * kGemmGroupW];
    __shared__ __attribute__((aligned(16))) bf16_t Xs[3 * 64 * kGemmPitch];
    bf16_t *const planes[3] = {Xs, Xs + 64 * kGemmPitch, Xs + 2 * 64 * kGemmPitch};
    gemm64<CW>(J, W, ldw, K, blockIdx.x, Ws, planes);
}

// ---------------------------------------------------------------------------
// The large products: a BM x BN tile per workgroup on 32x32x16 products, a wavefront with a quarter of it (BM / 2 x BN / 2), the contraction in chunks of 64 that go from memory straight into LDS (16 bytes per lane, no registers in
// between) into one of two buffers while the other is multiplied.
// A chunk's rows lie unpadded, as the direct loads need; conflicts are avoided by exchanging 16-byte pieces: piece c of
// row m of In sits at position c ^ (m % 8) (16-byte row reads of 8 rows then cover all banks), piece c of row k of W
// at c ^ 4 (k % 4) (BN = 128) or c ^ 4 (k / 2 % 2) (BN = 64), so that the 4 rows of a transposing read, and the 2
// column groups next to each other, meet different banks.
// The product is formed transposed (rows = outputs) with W's columns taken in the order that leaves a lane with two
// runs of 8 consecutive outputs of one row of In per 32 outputs (see the operand layouts in bra_mfma.hip).
// What bounds it (8192 x 768 x 2304, 128 x 128 tiles): direct loads alone 24 us (18 TB/s out of the L2s), products with
// their LDS reads alone 23, stores alone 9.5; they overlap to 37 (43.7 where the compiler counted the direct loads and a
// chunk past the end was loaded once more).
// BT: W is given transposed, [Nout][ldw] with the contraction axis contiguous; its chunk then lies like In's and needs no
// transposing reads.
alignas(16) __device__ bf16_t zero_row[4096];        // what missing rows of In read (never written)

// Row of the map in memory that row m of the padded map is, or -1.
__device__ __forceinline__ long stored_row(const GemmRows &r, int m)
{
    const int hw = r.Hp * r.Wp, b = m / hw, t = m - b * hw, y = t / r.Wp, x = t - y * r.Wp;
    return y < r.H && x < r.W ? ((long)b * r.H + y) * r.W + x : -1;
}

// LDS of a workgroup.  A single chunk: four workgroups per compute unit (with eight, 200704 x 64 x 64 takes 13.7 us instead of 12.9).
template <int BM, int BN, int NB>
constexpr size_t ring_bytes() { return NB == 1 ? 40 * 1024 : (size_t)NB * (BM + BN) * 64 * 2; }

// What lies in front of the table of rows of a product with means.
template <int BM, int BN, int NB>
__host__ __device__ constexpr size_t means_ring()
{
    constexpr size_t chunks = NB == 1 ? 38 * 1024 : (size_t)NB * (BM + BN) * 64 * 2, results = (size_t)BM * (BN + 4) * sizeof(float);
    return chunks > results ? chunks : results;
}

// Tokens of row `row` of tile `tile` of a product that goes region by region, in the map and in what is stored of it; -1: none.
template <int BM>
__device__ __forceinline__ void region_row(const GemmMeans &g, int tile, int row, int &token, int &stored)
{
    token = stored = -1;
    const int per = fast_div(BM, g.n_inv), first = tile * per, b0 = (unsigned)first / (unsigned)g.R, r0 = first - b0 * g.R;
    const int j = fast_div(row, g.n_inv), t = row - j * g.n;
    if (j >= per || first + j >= g.regions) return;
    const int over = fast_div(r0 + j, g.R_inv), reg = r0 + j - over * g.R;
    const int ry = fast_div(reg, g.S_inv), ty = fast_div(t, g.rw_inv);
    const int y = ry * g.rh + ty, x = (reg - ry * g.S) * g.rw + t - ty * g.rw;
    token = ((b0 + over) * g.S * g.rh + y) * g.S * g.rw + x;
    if (y < g.H && x < g.W) stored = ((b0 + over) * g.H + y) * g.W + x;
}

// How far the pieces of row `row` of a transposed W are turned: differently for the 8 rows that 8 lanes next to each other read, which
// differ in bits 0, 1 and 3 (see fragments()).
__device__ __forceinline__ int bt_turn(int row) { return row % 4 + row / 8 % 2 * 4; }

// Workgroups of an XCD take neighbouring tiles, the output tiles of the same rows one after the other (swizzled()).
// EXT: bias, GELU, residual or rows that are not in memory (GemmRows).  NB: buffers, 1 for K = 64, else 2.
// lds: NB chunks of In and of W.
// MEANS: rows region by region, see GemmMeans (M is not looked at); a table in LDS has the tokens of the tile's rows.  The float32 results of
// the columns that have means are added up over aligned groups of 16 or 4 rows in registers (means_group()), where that is less
// than a region the groups' sums, or with an odd number of rows the results, meet in LDS: the order does not depend on the tile.  All by way of
// LDS it took 1 us more of 64 x 14 x 14 x 384's layer (68.5 -> 67.0) and of 8 x 32 x 32 x 768's bra_route (39.2 -> 38.3).
template <int BM, int BN, int NB, bool BT, bool EXT, bool MEANS = false, bool BASED = false>
__device__ __forceinline__ void dma_tile(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw, int M, int K, int Nout,
                                         const GemmOut &out, int block, bf16_t *lds, const GemmMeans *means = nullptr)
{
    constexpr int AE = BM * 64, BE = BN * 64;     // elements of a chunk
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, h = lane / 32, c = lane % 32;
    const int otiles = (Nout + BN - 1) / BN;
    const int m0 = (block / otiles) * BM, o0 = (block % otiles) * BN;
    if (!MEANS && m0 >= M) return;                // the grid is rounded up to a multiple of 8
    const int *rows = nullptr;                    // tokens of the tile's rows, in the map and as stored
    if constexpr (MEANS) {
        if (block / otiles * fast_div(BM, means->n_inv) >= means->regions) return;
        int *table = (int *)((char *)lds + means_ring<BM, BN, NB>());
        if (tid < BM) region_row<BM>(*means, block / otiles, tid, table[tid], table[BM + tid]);
        __syncthreads();
        rows = table;
    }

    constexpr int LA = BM / 32, LB = BN / 32;     // direct loads of a wavefront per chunk
    // W by bytes from the chunk's first row, and with BASED In from the tile's.  Beside the region-level product of K >= 512 that is
    // faster (8 x 32 x 32 x 768: the launch 41 us for 47, the layer 108.7 -> 104.5; 16 x 21 x 35 x 512 88.9 -> 86.1), with K = 384 and less it is
    // not always (64 x 16 x 24 x 384 123.8 -> 125.7, 20 x 56 x 56 x 192 111.7 -> 110.6), alone it is slower (8 x 32 x 32 x 768 with a given index 96.7 ->
    // 100.8, gradients of 64 x 14 x 14 x 384 167 -> 176)
    const bf16_t *ap[LA], *abase = In + (size_t)(BASED ? m0 : 0) * K, *bbase = W;
    unsigned aoff[LA], boff[LB];
#pragma unroll
    for (int u = 0; u < LA; ++u) {
        const int row = 8 * (wave * LA + u) + lane / 8, piece = (lane % 8) ^ (row % 8);
        ap[u] = In + (size_t)(MEANS ? 0 : min(m0 + row, M - 1)) * K + 8 * piece;
        aoff[u] = 2 * ((min(m0 + row, M - 1) - m0) * K + 8 * piece);
        if constexpr (MEANS) {
            const int at = rows[BM + row];
            ap[u] = (at >= 0 ? In + (size_t)at * K : zero_row) + 8 * piece;
        } else if (EXT && out.in_rows.Hp) {
            const long at = stored_row(out.in_rows, min(m0 + row, M - 1));
            ap[u] = (at >= 0 ? In + (size_t)at * K : zero_row) + 8 * piece;
        }
    }
    constexpr int CH = BN / 8, RPI = 64 / CH;     // pieces of a row of W, rows per direct load
#pragma unroll
    for (int u = 0; u < LB; ++u) {
        if (BT) {
            const int row = 8 * (wave * LB + u) + lane / 8, piece = (lane % 8) ^ bt_turn(row);
            boff[u] = 2 * ((min(o0 + row, Nout - 1) - o0) * ldw + 8 * piece);
            continue;
        }
        const int k = RPI * (wave * LB + u) + lane / CH;
        const int piece = (lane % CH) ^ (BN == 128 ? 4 * (k % 4) : 4 * (k / 2 % 2));
        boff[u] = 2 * (k * ldw + min(o0 + 8 * piece, Nout - 8));
    }
    if (BT) bbase += (size_t)o0 * ldw;
    const unsigned base = lds_address(lds);
    auto request = [&](int chunk, int buffer) {
        const int k0 = 64 * chunk;
        const unsigned at = base + buffer * (AE + BE) * 2;
        lds_reads_done();
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            if (!BASED) load_to_lds_untracked(ap[u] + k0, at + 1024 * (wave * LA + u));
            else load_to_lds_untracked(abase + k0, aoff[u], at + 1024 * (wave * LA + u));
        }
#pragma unroll
        for (int u = 0; u < LB; ++u) load_to_lds_untracked(bbase + (BT ? (size_t)k0 : (size_t)k0 * ldw), boff[u], at + AE * 2 + 1024 * (wave * LB + u));
    };
    constexpr int MT = BM / 64, NT = BN / 64;     // 32 x 32 tiles of a wavefront
    const int wm = (wave / 2) * (BM / 2), wn = (wave % 2) * (BN / 2);
    f32x16 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[nt][mt][e] = 0.f;
    // transposing read of W: lane s of a 16-lane group q gives the address of 4 columns of row k; with the two middle
    // bits of the column exchanged (see above)
    const int s = lane % 16, q = lane / 16, col4 = ((s % 4) % 2) * 2 + (s % 4) / 2;
    auto fragments = [&](const bf16_t *As, const bf16_t *Bs, int ks, bf16x8 (&xf)[MT], bf16x8 (&wf)[NT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int row = wm + 32 * mt + c;
            xf[mt] = *(const bf16x8 *)(As + row * 64 + 8 * ((2 * ks + h) ^ (row % 8)));
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (BT) {
                // operand row c is output c with its two middle bits exchanged
                const int row = wn + 32 * nt + (c & 0x13) + ((c & 4) << 1) + ((c & 8) >> 1);
                wf[nt] = *(const bf16x8 *)(Bs + row * 64 + 8 * ((2 * ks + h) ^ bt_turn(row)));
                continue;
            }
            u32x2 r[2];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int k = 16 * ks + 8 * (q / 2) + 4 * half + s / 4;
                const int o = wn + 32 * nt + 16 * (q % 2) + 4 * col4, piece = o / 8;
                const int pos = piece ^ (BN == 128 ? 4 * (k % 4) : 4 * (k / 2 % 2));
                r[half] = __builtin_bit_cast(u32x2, lds_read_tr16(Bs + k * BN + 8 * pos + o % 8));
            }
            wf[nt] = __builtin_bit_cast(bf16x8, u32x4{r[0][0], r[0][1], r[1][0], r[1][1]});
        }
    };
    // the next step's operands are on their way while this step's products run
    auto multiply = [&](const bf16_t *As, const bf16_t *Bs) {
        bf16x8 xf[2][MT], wf[2][NT];
        fragments(As, Bs, 0, xf[0], wf[0]);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) fragments(As, Bs, ks + 1, xf[(ks + 1) % 2], wf[(ks + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = mfma32(wf[ks % 2][nt], xf[ks % 2][mt], acc[nt][mt]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int chunks = NB == 1 ? 1 : K / 64;
    request(0, 0);
    for (int c0 = 0; c0 < chunks; c0 += NB) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if (c0 + u >= chunks) break;
            arrive_barrier();                      // the chunk has arrived; the other buffer has been read
            if (NB > 1 && c0 + u + 1 < chunks) request(c0 + u + 1, 1 - u);
            multiply(lds + u * (AE + BE), lds + u * (AE + BE) + AE);
        }
    }
    products_done();
    constexpr int MP = BN + 4;                    // floats per row of sums in LDS
    const bool averaged = MEANS && o0 < 2 * out.cols;
    float *sums = (float *)lds;
    if constexpr (MEANS) {
        auto lay_down = [&](auto group) {
            constexpr int G = decltype(group)::value;
            const bool whole = G == means->n;
            if (!whole) __syncthreads();          // the last chunk has been read
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int ot = __builtin_amdgcn_readfirstlane(o0 + wn + 32 * nt), which = (ot >= out.cols) + (ot >= 2 * out.cols);
                float *to = which < 2 ? means->buf[which] + ot - which * out.cols : nullptr;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int row = wm + 32 * mt + c;
                    if constexpr (G == 1) {
#pragma unroll
                        for (int e = 0; e < 16; e += 4)
                            *(f32x4 *)(sums + row * MP + wn + 32 * nt + 8 * h + 16 * (e / 8) + e % 8) = f32x4{acc[nt][mt][e], acc[nt][mt][e + 1], acc[nt][mt][e + 2], acc[nt][mt][e + 3]};
                        continue;
                    }
                    f32x4 quad = quad_sums(acc[nt][mt], c);
                    if constexpr (G == 16)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            quad[e] += dpp_get<0x124>(quad[e]);       // row_ror:4
                            quad[e] += dpp_get<0x128>(quad[e]);       // row_ror:8
                        }
                    if (c % G >= 4) continue;
                    const int col = 8 * h + 16 * (c % 2) + 4 * (c / 2 % 2);
                    const int region = block / otiles * (BM / G) + row / G;
                    if (!whole) *(f32x4 *)(sums + row / G * MP + wn + 32 * nt + col) = quad;
                    else if (to && region < means->regions) *(f32x4 *)(to + (size_t)region * out.cols + col) = quad * means->n_inv;
                }
            }
        };
        if (averaged) {
            const int G = means_group(means->n);
            if (G == 16) lay_down(std::integral_constant<int, 16>{});
            else if (G == 4) lay_down(std::integral_constant<int, 4>{});
            else lay_down(std::integral_constant<int, 1>{});
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        // a 32-output tile lies in one buffer (cols is a multiple of 32): looked up once per tile, for the whole wavefront
        const int ot = __builtin_amdgcn_readfirstlane(o0 + wn + 32 * nt);
        if (ot >= Nout) continue;                  // of no buffer
        const int which = (ot >= out.cols) + (ot >= 2 * out.cols), ct = ot - which * out.cols;
        bf16_t *buf = (bf16_t *)out.buf[which];
        if (MEANS && !buf) continue;
        float *fbuf = which < 2 ? out.f32[which] : nullptr;
        const float scale = which == 0 ? out.scale0 : 1.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = MEANS ? rows[wm + 32 * mt + c] : m0 + wm + 32 * mt + c;
            if (MEANS ? m < 0 : m >= M) continue;
            size_t row = (size_t)m * out.cols;
            if (EXT && out.out_rows.Hp) {
                const long at = stored_row(out.out_rows, m);
                if (at < 0) continue;
                row = (size_t)at * out.cols;
            }
#pragma unroll
            for (int run = 0; run < 2; ++run) {
                const int o = ot + 16 * run + 8 * h, col = ct + 16 * run + 8 * h;
                if (o >= Nout) continue;
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = acc[nt][mt][8 * run + e];
                if (fbuf) {
                    *(f32x4 *)(fbuf + row + col) = f32x4{v[0], v[1], v[2], v[3]};
                    *(f32x4 *)(fbuf + row + col + 4) = f32x4{v[4], v[5], v[6], v[7]};
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] *= scale;
                if (EXT) {
                    if (out.bias) {
                        const f32x4 b0 = *(const f32x4 *)(out.bias + o), b1 = *(const f32x4 *)(out.bias + o + 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { v[e] += b0[e]; v[4 + e] += b1[e]; }
                    }
                    if (out.gelu) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = gelu_f32(v[e]);
                    }
                    if (out.res) {
                        const u32x4 rv = *(const u32x4 *)(out.res + row + o);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { v[2 * e] += bf16_lo(rv[e]); v[2 * e + 1] += bf16_hi(rv[e]); }
                    }
                }
                *(bf16x8 *)(buf + row + col) = pack8(v);
            }
        }
    }
    if constexpr (MEANS) {
        const int n = means->n, G = means_group(n), per = fast_div(BM, means->n_inv), rows_each = n / G;
        if (!averaged || G == n) return;
        __syncthreads();
        constexpr int GROUPS = BN / 4, TR = 256 / GROUPS;
        const int col = o0 + 4 * (tid % GROUPS), which = (col >= out.cols) + (col >= 2 * out.cols);
        const int first = block / otiles * per;
        for (int j = tid / GROUPS; j < per && first + j < means->regions; j += TR) {
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
            const float *p = sums + j * rows_each * MP + 4 * (tid % GROUPS);
#pragma unroll 4
            for (int t = 0; t < rows_each; ++t) sum += *(const f32x4 *)(p + t * MP);
            if (which < 2) *(f32x4 *)(means->buf[which] + (size_t)(first + j) * out.cols + col - which * out.cols) = sum * means->n_inv;
        }
    }
}

template <int BM, int BN, int NB, bool REGIONS, bool BT, bool EXT, bool BASED>
__global__ __launch_bounds__(256, BM == 64 && BN == 64 ? 3 : 2) void k_gemm_dma(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw,
                                                  int M, int K, int Nout, GemmOut out, GemmRegions reg, int reg_blocks)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *lds = (bf16_t *)smem;
    if (REGIONS && (int)blockIdx.x < reg_blocks) {
        bf16_t *const planes[3] = {lds, lds + 64 * kGemmPitch, lds + 2 * 64 * kGemmPitch};
        gemm64<2>(reg, W, ldw, K, blockIdx.x, lds + 3 * 64 * kGemmPitch, planes);
        return;
    }
    dma_tile<BM, BN, NB, BT, EXT, false, BASED>(In, W, ldw, M, K, Nout, out, swizzled((int)blockIdx.x - reg_blocks, (int)gridDim.x - reg_blocks), lds);
}

template <int BM, int BN, int NB>
__global__ __launch_bounds__(256, BM == 64 && BN == 64 ? 3 : 2) void k_gemm_means(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw,
                                                  int K, int Nout, GemmOut out, GemmMeans means)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    dma_tile<BM, BN, NB, false, false, true>(In, W, ldw, 0, K, Nout, out, swizzled_block(), (bf16_t *)smem, &means);
}

// Two products over the same rows and contraction in one launch: Q, K, V = X Wqkv and dO = dY Wo^T (W transposed).  12544 x 384:
// 24.1 us, 29.8 as two launches; 2048 x 768 13.1 and 23.
template <int BM, int BN, int NB>
__global__ __launch_bounds__(256, BM == 64 && BN == 64 ? 3 : 2) void k_gemm_pair(const bf16_t *__restrict__ In0, const bf16_t *__restrict__ W0, int ldw0, int Nout0,
                                                  GemmOut out0, const bf16_t *__restrict__ In1, const bf16_t *__restrict__ W1, int ldw1, int Nout1,
                                                  GemmOut out1, int M, int K, int blocks0)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bi = blockIdx.x;
    if (bi < blocks0) dma_tile<BM, BN, NB, false, false>(In0, W0, ldw0, M, K, Nout0, out0, swizzled(bi, blocks0), (bf16_t *)smem);
    else dma_tile<BM, BN, NB, true, false>(In1, W1, ldw1, M, K, Nout1, out1, swizzled(bi - blocks0, (int)gridDim.x - blocks0), (bf16_t *)smem);
}

long region_blocks(const GemmRegions &r) { return (r.M + 63) / 64 * ((r.Nout + 63) / 64); }

template <int BM, int BN>
long tile_blocks(long M, int Nout) { return ((M + BM - 1) / BM * ((Nout + BN - 1) / BN) + 7) / 8 * 8; }

template <typename K>
bool opt_in(K kernel, bool &done)
{
    if (!done) done = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) == hipSuccess;
    return done;
}

template <int BM, int BN, int NB, bool REGIONS, bool BT, bool EXT, bool BASED = false>
int launch_dma_t(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out,
               const GemmRegions &reg, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_gemm_dma<BM, BN, NB, REGIONS, BT, EXT, BASED>, opted)) return BRA_ERR_LAUNCH;
    const long blocks = tile_blocks<BM, BN>(M, Nout);
    const long rb = REGIONS ? region_blocks(reg) : 0;
    if (blocks + rb > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((k_gemm_dma<BM, BN, NB, REGIONS, BT, EXT, BASED>), dim3((unsigned)(blocks + rb)), dim3(256),
                       std::max(ring_bytes<BM, BN, NB>(), REGIONS ? kGemm64Bytes : 0), st, In, W, ldw, (int)M, K, Nout, out, reg, (int)rb);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

template <int BM, int BN, int NB, bool REGIONS, bool BT>
int launch_dma(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out,
               const GemmRegions &reg, hipStream_t st)
{
    if constexpr (!BT) {
        if (out.bias || out.gelu || out.res || out.in_rows.Hp || out.out_rows.Hp)
            return launch_dma_t<BM, BN, NB, REGIONS, false, true>(In, W, ldw, M, K, Nout, out, reg, st);
    }
    if constexpr (REGIONS && BM == 128) {
        if (K >= 512) return launch_dma_t<BM, BN, NB, true, BT, false, true>(In, W, ldw, M, K, Nout, out, reg, st);
    }
    return launch_dma_t<BM, BN, NB, REGIONS, BT, false>(In, W, ldw, M, K, Nout, out, reg, st);
}

template <int BM, int BN, int NB>
int launch_means(const bf16_t *In, const bf16_t *W, int ldw, int K, int Nout, const GemmOut &out, const GemmMeans &means, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_gemm_means<BM, BN, NB>, opted)) return BRA_ERR_LAUNCH;
    const long blocks = (((long)means.regions + BM / means.n - 1) / (BM / means.n) * ((Nout + BN - 1) / BN) + 7) / 8 * 8;
    if (blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((k_gemm_means<BM, BN, NB>), dim3((unsigned)blocks), dim3(256), (means_ring<BM, BN, NB>() + 2 * BM * sizeof(int)), st, In, W, ldw, K, Nout, out,
                       means);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

enum Tile { kOneChunk, kWide, kMid, kNarrow };

// One chunk: no tile reads anything twice, small ones overlap their loads and stores best (126464 x 64 x 192: 14.0 us, 14.8
// with 64 x 128, 15.6 with 128 x 128).
// Wide tiles read less per product, narrow ones deal out more evenly over the 256 compute units.  Time is that of the
// compute unit with the most tiles: 744, 433 or 260 for one of 128 x 128, 64 x 128 or 64 x 64 (12544 x 768 x 2304:
// 52.1, 60.7 and 71.1 us for 7, 14 and 28 tiles), three tenths more where it has a single one and nothing to overlap it
// with.  Measured, 128 x 128 / 64 x 128 / 64 x 64 (us): 8192 x 768 x 2304: 37.2 / 38.9 / 47.1; 8192 x 768 x 768: 15.9 / 14.6 /
// 17.1; 12544 x 1152 x 384: 20.8 / 19.3 / 21.9; 12544 x 512 x 512: 12.4 / 14.0 / 12.7; 3136 x 768 x 768: 9.9 / 9.3 / 8.3;
// 12544 x 256 x 768: 12.2 / 11.2 / 12.0; 1568 x 384 x 1152: 6.6 / 5.2 / 4.8.  A third buffer, 256 x 128 tiles with 8 wavefronts
// and chunks of 32 gained nothing.
// Nout1: columns of a second product over the same rows.  others: workgroups of a region-level product in the launch, each as
// long as a 64 x 128 tile (32 x 16 x 16 x 768, 768 of them: 64 x 128 tiles, a layer in 129.7 us, for 128 x 128, 133.6; 8 x 32 x 32 x 768,
// 192 of them: 128 x 128, 107.2, for 64 x 128, 109.8).
// Weights that an XCD's 4 MB L2 does not hold come in again for every row tile: a tenth more for tiles of 64 rows, from 40 of them on
// (4900 x 1024 x 3072 with its regions 66.6 / 77.8 / 87.8, 3920 x 1024 x 3072 52.9 / 58.6 / 66.1, 3920 x 1280 x 3840 80 / 106 / 112; but 4900 x
// 3072 x 1024 52.5 / 49.0, and 1960 x 1024 x 3072 33.5 / 31.2).
// Up to three chunks and one and a half wide tiles of columns: the wide tile's empty half is a quarter of a short product
// (125440 x 192 x 192 25.3 / 26.3 / 23.8, 50176 13.4 / 13.6 / 12.4).
// n: rows in tiles of whole groups of n.
Tile pick_tile(long M, int K, int Nout, int Nout1, long others, int n = 1)
{
    if (K == 64) return kOneChunk;
    if (K <= 192 && Nout > 128 && Nout + Nout1 <= 192) return kNarrow;
    auto cost = [&](int bm, int bn, long tile) {
        const long groups = bm / n, row_tiles = (M / n + groups - 1) / groups;
        const long rounds = (row_tiles * ((Nout + bn - 1) / bn + (Nout1 + bn - 1) / bn) + others * 433 / tile + 255) / 256;
        return tile * rounds * (rounds == 1 ? 13 : 10);
    };
    const bool again = (long)K * Nout * 2 > 4L << 20 && M > 2560;
    const long wide = cost(128, 128, 744), mid = cost(64, 128, again ? 476 : 433), narrow = cost(64, 64, again ? 286 : 260);
    return wide <= mid && wide <= narrow ? kWide : mid <= narrow ? kMid : kNarrow;
}

template <bool REGIONS, bool BT = false>
int launch_big(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out, const GemmRegions &reg,
               hipStream_t st)
{
    switch (pick_tile(M, K, Nout, 0, REGIONS ? region_blocks(reg) : 0)) {
    case kOneChunk: return launch_dma<64, 64, 1, REGIONS, BT>(In, W, ldw, M, K, Nout, out, reg, st);
    case kWide: return launch_dma<128, 128, 2, REGIONS, BT>(In, W, ldw, M, K, Nout, out, reg, st);
    case kMid: return launch_dma<64, 128, 2, REGIONS, BT>(In, W, ldw, M, K, Nout, out, reg, st);
    default: return launch_dma<64, 64, 2, REGIONS, BT>(In, W, ldw, M, K, Nout, out, reg, st);
    }
}

// Few rows: a tile of 32 rows x 32 outputs per workgroup, whose wavefronts share the contraction and add up through LDS in a fixed order.  The tiles
// above leave most of the chip idle there and walk the whole contraction a chunk of 64 at a time, each 0.5 us of latency (128 x 2304 x 768:
// 18 us on 24 workgroups).  A wavefront brings its steps of 32 by itself, both operands straight into its own ring of kSplitAhead steps, 64 bytes per
// row; there is no barrier before the sums.  In's pieces of 16 bytes are exchanged (piece p of row r at p ^ (r / 4 % 4)): rows 4 apart meet
// different banks.  W as above, its columns in order.  Nout and out.cols are multiples of 32; MEANS: n <= 32.
constexpr int kSplitAhead = 3, kSplitPitch = 36;       // floats per row of sums
template <int WAVES>
constexpr size_t split_bytes()
{
    constexpr size_t ring = (size_t)WAVES * kSplitAhead * 4096, sums = (size_t)WAVES * 32 * kSplitPitch * 4;
    return (ring > sums ? ring : sums) + 2 * 32 * sizeof(int);
}

template <bool BT, bool MEANS, int WAVES>
__device__ __forceinline__ void split_tile(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw, int M, int K, int Nout, const GemmOut &out,
                                           int block, char *smem, const GemmMeans *means = nullptr)
{
    constexpr int P = kSplitPitch, AHEAD = kSplitAhead;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, h = lane / 32, c = lane % 32;
    const int ntiles = Nout / 32, tile = block / ntiles, n0 = 32 * (block - tile * ntiles), m0 = 32 * tile;
    int *table = (int *)(smem + split_bytes<WAVES>() - 2 * 32 * sizeof(int));       // MEANS: tokens of the tile's rows
    if constexpr (MEANS) {
        if (tid < 32) region_row<32>(*means, tile, tid, table[tid], table[32 + tid]);
        __syncthreads();
    }
    const int steps = K / 32, s0 = steps * wave / WAVES, s1 = steps * (wave + 1) / WAVES;
    // direct loads: 16 rows of 4 pieces each
    const bf16_t *x[2], *w[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row = 16 * u + lane / 4, piece = (lane % 4) ^ (row / 4 % 4);
        const long at = MEANS ? (long)table[32 + row] : out.in_rows.Hp ? stored_row(out.in_rows, min(m0 + row, M - 1)) : (long)min(m0 + row, M - 1);
        x[u] = (at >= 0 ? In + (size_t)at * K : zero_row) + 8 * piece;
        if (BT) w[u] = W + (size_t)(n0 + row) * ldw + 8 * piece;
        else w[u] = W + (size_t)row * ldw + n0 + 8 * (lane % 4);
    }
    const size_t wstep = BT ? 32 : (size_t)32 * ldw;
    char *ring = smem + wave * AHEAD * 4096;
    const unsigned base = lds_address(ring);
    auto request = [&](int s, int slot) {
        lds_reads_done();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            load_to_lds_untracked(x[u] + 32 * s, base + 4096 * slot + 1024 * u);
            load_to_lds_untracked(w[u] + s * wstep, base + 4096 * slot + 2048 + 1024 * u);
        }
    };
    const int sl = lane % 16, q = lane / 16;
    auto row_operand = [&](const bf16_t *T, int ks) { return *(const bf16x8 *)(T + c * 32 + 8 * ((2 * ks + h) ^ (c / 4 % 4))); };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (s0 + a < s1) request(s0 + a, a);
    for (int s = s0; s < s1; s += AHEAD) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
            if (s + a >= s1) break;
            const int behind = s1 - 1 - s - a;     // steps requested after this one: four loads each
            if (behind >= 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else if (behind == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const bf16_t *X = (const bf16_t *)(ring + 4096 * a), *B = X + 1024;
            bf16x8 xf[2], wf[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                xf[ks] = row_operand(X, ks);
                if (BT) {
                    wf[ks] = row_operand(B, ks);
                } else {
                    u32x2 r[2];
#pragma unroll
                    for (int half = 0; half < 2; ++half)
                        r[half] = __builtin_bit_cast(u32x2, lds_read_tr16(B + (16 * ks + 8 * (q / 2) + 4 * half + sl / 4) * 32 + 16 * (q % 2) + 4 * (sl % 4)));
                    wf[ks] = __builtin_bit_cast(bf16x8, u32x4{r[0][0], r[0][1], r[1][0], r[1][1]});
                }
            }
            if (s + a + AHEAD < s1) request(s + a + AHEAD, a);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) acc = mfma32(wf[ks], xf[ks], acc);
        }
    }
    products_done();
    __syncthreads();                              // every ring has been read
    float *sums = (float *)smem;
#pragma unroll
    for (int e = 0; e < 16; e += 4) *(f32x4 *)(sums + (wave * 32 + c) * P + 2 * e + 4 * h) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
    __syncthreads();
    const int which = (n0 >= out.cols) + (n0 >= 2 * out.cols), col0 = n0 - which * out.cols;
    bf16_t *buf = (bf16_t *)out.buf[which];
    float *fbuf = which < 2 ? out.f32[which] : nullptr;
    const float scale = which == 0 ? out.scale0 : 1.0f;
    if (tid < 256) {                              // (row, 4 outputs)
        const int row = tid / 8, col = 4 * (tid % 8);
        float *at = sums + row * P + col;
        f32x4 v = *(const f32x4 *)at;
#pragma unroll
        for (int u = 1; u < WAVES; ++u) v += *(const f32x4 *)(at + u * 32 * P);
        if (MEANS) *(f32x4 *)at = v;
        const int m = MEANS ? table[row] : m0 + row;
        const long to = (MEANS ? m < 0 : m >= M) || !buf ? -1 : out.out_rows.Hp ? stored_row(out.out_rows, m) : m;
        if (to >= 0) {
            const size_t o = (size_t)to * out.cols + col0 + col;
            if (fbuf) *(f32x4 *)(fbuf + o) = v;
            v *= scale;
            if (out.bias) v += *(const f32x4 *)(out.bias + n0 + col);
            if (out.gelu) v = f32x4{gelu_f32(v[0]), gelu_f32(v[1]), gelu_f32(v[2]), gelu_f32(v[3])};
            if (out.res) {
                const u32x2 r = *(const u32x2 *)(out.res + (size_t)to * out.cols + n0 + col);
                v += f32x4{bf16_lo(r[0]), bf16_hi(r[0]), bf16_lo(r[1]), bf16_hi(r[1])};
            }
            *(u32x2 *)(buf + o) = pack4(v);
        }
    }
    if constexpr (MEANS) {
        if (which >= 2) return;
        __syncthreads();
        const int n = means->n, per = fast_div(32, means->n_inv), first = tile * per;
        for (int e = tid; e < 8 * per; e += 64 * WAVES) {
            const int j = e / 8;
            if (first + j >= means->regions) break;
            const float *at = sums + j * n * P + 4 * (e % 8);
            f32x4 sum = *(const f32x4 *)at;
            for (int t = 1; t < n; ++t) sum += *(const f32x4 *)(at + t * P);
            *(f32x4 *)(means->buf[which] + (size_t)(first + j) * out.cols + col0 + 4 * (e % 8)) = sum * means->n_inv;
        }
    }
}

constexpr int kSplitWaves = 8;

__global__ __launch_bounds__(64 * kSplitWaves) void k_gemm_split(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw, int M, int K, int Nout,
                                                                 GemmOut out)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    split_tile<false, false, kSplitWaves>(In, W, ldw, M, K, Nout, out, blockIdx.x, smem);
}

__global__ __launch_bounds__(64 * kSplitWaves) void k_gemm_means_split(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw, int K, int Nout,
                                                                       GemmOut out, GemmMeans means)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    split_tile<false, true, kSplitWaves>(In, W, ldw, 0, K, Nout, out, blockIdx.x, smem, &means);
}

__global__ __launch_bounds__(64 * kSplitWaves) void k_gemm_pair_split(const bf16_t *__restrict__ In0, const bf16_t *__restrict__ W0, int ldw0, int Nout0, GemmOut out0,
                                                                      const bf16_t *__restrict__ In1, const bf16_t *__restrict__ W1, int ldw1, int Nout1,
                                                                      GemmOut out1, int M, int K, int blocks0)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bi = blockIdx.x;
    if (bi < blocks0) split_tile<false, false, kSplitWaves>(In0, W0, ldw0, M, K, Nout0, out0, bi, smem);
    else split_tile<true, false, kSplitWaves>(In1, W1, ldw1, M, K, Nout1, out1, bi - blocks0, smem);
}

long split_blocks(long M, int Nout) { return (M + 31) / 32 * (Nout / 32); }

// blocks: the workgroups it would take.  A round of them, one per compute unit (98 KB of LDS), takes about 4 us; tiles of 64 x 64 take 0.5 us for 64 of the
// contraction, so that a short one leaves nothing to gain and only a long one pays for a second round.  Blocks, tiles of 64 / split (us, whole calls): gradients of
// 1 x 7 x 7 x 512 34.1 / 27.0, of 2 x 7 x 7 x 768 46.8 / 38.1; block of 2 x 8 x 8 x 768 73.7 / 60.3, of 1 x 14 x 14 x 384 45.9 / 40.7; K = 256, forward of 6 x 7 x 7 x 256 (240) 19.9 / 18.8,
// 8 x 7 x 7 x 256 (312) 20.1 / 20.6, 2 x 14 x 14 x 256 (312) 21.1 / 22.5, 2 x 16 x 16 x 256 (384) 19.4 / 22.5; K = 384, 4 x 7 x 7 x 384 (252) 23.2 / 20.3, 1 x 14 x 21 x 384 (360) 23.7 / 24.1;
// K = 2304, gradients of 2 x 14 x 14 x 768 (312) 49.1 / 44.0; K = 192, gradients of 2 x 24 x 24 x 192 29.8 / 31.9.
bool splits(long blocks, int K, int Nout, int cols)
{
    return Nout % 32 == 0 && cols % 32 == 0 && blocks <= (K >= 1024 ? 512 : K >= 256 ? 256 : 0);
}

int launch_split(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_gemm_split, opted)) return BRA_ERR_LAUNCH;
    hipLaunchKernelGGL(k_gemm_split, dim3((unsigned)split_blocks(M, Nout)), dim3(64 * kSplitWaves), split_bytes<kSplitWaves>(), st, In, W, ldw, (int)M, K, Nout, out);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

template <int BM, int BN, int NB>
int launch_pair(const GemmHalf &a, const GemmHalf &b, long M, int K, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_gemm_pair<BM, BN, NB>, opted)) return BRA_ERR_LAUNCH;
    const long b0 = tile_blocks<BM, BN>(M, a.Nout), b1 = tile_blocks<BM, BN>(M, b.Nout);
    if (b0 + b1 > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((k_gemm_pair<BM, BN, NB>), dim3((unsigned)(b0 + b1)), dim3(256), (ring_bytes<BM, BN, NB>()), st, a.In, a.W, a.ldw, a.Nout, a.out,
                       b.In, b.W, b.ldw, b.Nout, b.out, (int)M, K, (int)b0);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// ---------------------------------------------------------------------------
// PAIR: the workgroup also holds a K x K matrix W1, given transposed, and forms Out1 = In1 W1^T for its rows (Q, K, V and dO of the
// backward pass; 64 x 56 x 56 x 64: 35.5 us for 39 in two launches, 25088 x 128: 24.9 for 29).
template <int K, int N, bool PAIR>
__global__ __launch_bounds__(1024) void k_proj(const bf16_t *__restrict__ In, const bf16_t *__restrict__ W, int ldw, long M,
                                               int per_group, GemmOut out, const bf16_t *__restrict__ In1, const bf16_t *__restrict__ W1, int ldw1, GemmOut out1)
{
    constexpr int KS = K / 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *Ws = (bf16_t *)smem, *W1s = (bf16_t *)(smem + ProjLds<K, N, false>::bytes);
    const int T = blockDim.x, tid = threadIdx.x, waves = T / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, g = lane / 16, i = lane % 16;
    const long tiles = (M + 15) / 16, first = (long)blockIdx.x * per_group, last = min(tiles, first + per_group);
    bf16x8 x[2][KS], y[2][KS];
    auto fetch = [&](long tile, int set) {
        const size_t row = (size_t)min(min(tile, tiles - 1) * 16 + i, M - 1) * K + 8 * g;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            x[set][ks] = *(const bf16x8 *)(In + row + 32 * ks);
            if (PAIR) y[set][ks] = *(const bf16x8 *)(In1 + row + 32 * ks);
        }
    };
    fetch(first + wave, 0);
    proj_stage<K, N, false>(Ws, W, ldw);
    if (PAIR) proj_stage<K, K, true>(W1s, W1, ldw1);
    __syncthreads();
    int again = 0;
    auto work = [&](long t, int set) {
        asm volatile("" : "+s"(again));
        proj_tile<K, N, false>(Ws, again, x[set], t, M, out);
        if (PAIR) proj_tile<K, K, true>(W1s, again, y[set], t, M, out1);
    };
    for (long t = first + wave; t < last; t += 2 * waves) {
        fetch(t + waves, 1);
        work(t, 0);
        if (t + waves >= last) break;
        fetch(t + 2 * waves, 0);
        work(t + waves, 1);
    }
}

template <int K, int N, bool PAIR = false>
int launch_proj_t(const bf16_t *In, const bf16_t *W, int ldw, long M, const GemmOut &out, hipStream_t st, const GemmHalf &second = GemmHalf{})
{
    static bool opted = false;
    if (!opt_in(k_proj<K, N, PAIR>, opted)) return BRA_ERR_LAUNCH;
    // as many wavefronts as deal out a compute unit's share of the tiles in even rounds
    const long tiles = (M + 15) / 16, per = (tiles + 255) / 256, rounds = (per + 15) / 16;
    const int waves = (int)std::max(4L, (per + rounds - 1) / rounds);
    hipLaunchKernelGGL((k_proj<K, N, PAIR>), dim3((unsigned)((tiles + per - 1) / per)), dim3(64 * waves),
                       (ProjLds<K, N, false>::bytes + (PAIR ? ProjLds<K, K, true>::bytes : 0)), st, In, W, ldw, M, (int)per, out, second.In, second.W,
                       second.ldw, second.out);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// Measured against the tiles (us): 50176 x 64 x 192 8.0 for 8.8, 200704 x 64 x 192 27 for 31; 25088 x 128 x 384 11.9 for 10.8,
// 50176 x 128 x 384 16.7 for 21.2, 150528 x 128 x 384 38.8 for 55.1; 50176 x 128 x 128 9.1 for 10.1; 64 x 64 no difference.
// The region-level product takes a launch of its own then, which K = 64 does not win back and K = 128 from about 100000 rows
// on (whole forward, 58800 rows: 79.8 -> 82.9; 283392 rows: 316 -> 298).
bool proj_ok(long M, int K, int N, const GemmOut &out, bool regions)
{
    const bool shape = K == 128 ? N == K || N == 3 * K : K == 64 && N == 3 * K && !regions;
    return shape && out.cols == K && M >= (regions ? 100000 : 40000) && !out.bias && !out.gelu && !out.res && !out.f32[0] && !out.f32[1] &&
           !out.in_rows.Hp && !out.out_rows.Hp;
}

int launch_proj(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int N, const GemmOut &out, hipStream_t st)
{
    if (K == 64) return launch_proj_t<64, 192>(In, W, ldw, M, out, st);
    return N == K ? launch_proj_t<128, 128>(In, W, ldw, M, out, st) : launch_proj_t<128, 384>(In, W, ldw, M, out, st);
}

// ---------------------------------------------------------------------------
// Part[share][a][n] = sum over the share's tokens t of A[t][a] B[t][n] (the weight gradients dWqkv = X^T dQKV and
// dWo = O^T dY, both in one launch): a 128 x 128 block of the output per workgroup, 64 tokens at a time straight into one of
// two LDS buffers; both operands by transposing reads (pieces exchanged as for W above).
// Bound by the loads: a share's rows are read by all blocks of it, 236 MB for 58 of 64 x 14 x 14 x 384.  All blocks of a share on one XCD, loads that
// the compiler does not count and no address arithmetic beyond a base per chunk: 36.5 -> 22 us (29 with the XCD's blocks alone;
// the matrix instructions take 7).  A ring of four buffers of 32 tokens was no faster, one workgroup per compute unit with four of 64 31.
constexpr int kTnTokens = 64;
constexpr size_t kTnBytes = (size_t)2 * 2 * kTnTokens * 128 * 2;

// block: of `blocks` (a multiple of 8), those of both products of a share one after the other, so that an XCD's L2 has the rows of its
// shares.
__device__ __forceinline__ void tn_block(const GemmTn &J0, const GemmTn &J1, int block, int blocks, long M, int share_tokens, bf16_t *lds)
{
    auto blocks_of = [](const GemmTn &J) { return ((J.N + 127) / 128) * ((J.KA + 127) / 128); };
    const int first = blocks_of(J0), each = first + blocks_of(J1), at = swizzled(block, blocks), share = at / each, rest = at - share * each;
    const GemmTn &J = rest < first ? J0 : J1;
    block = rest < first ? rest : rest - first;
    constexpr int TOK = kTnTokens, LOADS = TOK / 16;       // direct loads of each operand, by a wavefront
    const int nb = (J.N + 127) / 128;
    const int n0 = 128 * (block % nb), a0 = 128 * (block / nb);
    const long t_begin = (long)share * share_tokens, t_end = min(M, t_begin + share_tokens);
    if (t_begin >= M) return;                     // the grid is rounded up
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, h = lane / 32, c = lane % 32;
    const int ldl = lane / 16;                                // row of a direct load (4 rows of 16 pieces)
    const int piece = (lane % 16) ^ (4 * (ldl % 4));
    const int row0 = 4 * wave * LOADS + ldl, acol = min(a0 + 8 * piece, J.KA - 8), bcol = min(n0 + 8 * piece, J.N - 8);
    const bf16_t *abase = J.A + t_begin * J.lda, *bbase = J.Bm + t_begin * J.ldb;
    unsigned aoff[LOADS], boff[LOADS];            // bytes from the chunk's first row
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        aoff[u] = 2 * ((row0 + 4 * u) * J.lda + acol);
        boff[u] = 2 * ((row0 + 4 * u) * J.ldb + bcol);
    }
    const unsigned base = lds_address(lds) + 1024 * LOADS * wave;
    // the chunks one after the other: the bases move along
    auto request = [&](int chunk) {
        const unsigned at = base + chunk % 2 * (2 * TOK * 128 * 2);
        lds_reads_done();
        const int there = (int)min((long)TOK, t_end - t_begin - (long)TOK * chunk);      // rows; beyond, the last one is repeated
        if (there < TOK)
#pragma unroll
            for (int u = 0; u < LOADS; ++u) {
                aoff[u] = 2 * (min(row0 + 4 * u, there - 1) * J.lda + acol);
                boff[u] = 2 * (min(row0 + 4 * u, there - 1) * J.ldb + bcol);
            }
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            load_to_lds_untracked(abase, aoff[u], at + 1024 * u);
            load_to_lds_untracked(bbase, boff[u], at + TOK * 128 * 2 + 1024 * u);
        }
        abase += (size_t)TOK * J.lda;
        bbase += (size_t)TOK * J.ldb;
    };
    const int wa = (wave / 2) * 64, wn = (wave % 2) * 64;
    f32x16 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
    const int s = lane % 16, q = lane / 16;
    auto operand = [&](const bf16_t *T, int col0, int ks) {
        u32x2 r[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int k = 16 * ks + 8 * (q / 2) + 4 * half + s / 4, o = col0 + 16 * (q % 2) + 4 * (s % 4);
            r[half] = __builtin_bit_cast(u32x2, lds_read_tr16(T + k * 128 + 8 * ((o / 8) ^ (4 * (k % 4))) + o % 8));
        }
        return __builtin_bit_cast(bf16x8, u32x4{r[0][0], r[0][1], r[1][0], r[1][1]});
    };
    auto multiply = [&](const bf16_t *As, const bf16_t *Bs) {
        bf16x8 af[2][2], bf[2][2];
        auto fragments = [&](int ks) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                af[ks % 2][x] = operand(As, wa + 32 * x, ks);
                bf[ks % 2][x] = operand(Bs, wn + 32 * x, ks);
            }
        };
        fragments(0);
#pragma unroll
        for (int ks = 0; ks < TOK / 16; ++ks) {
            if (ks + 1 < TOK / 16) fragments(ks + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[x][y] = mfma32(af[ks % 2][x], bf[ks % 2][y], acc[x][y]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int chunks = (int)((t_end - t_begin + TOK - 1) / TOK);
    request(0);
    for (int k = 0; k < chunks; ++k) {
        arrive_barrier();                          // the chunk has arrived; the other buffer has been read
        if (k + 1 < chunks) request(k + 1);
        bf16_t *As = lds + k % 2 * (2 * TOK * 128);
        // tokens past the end add nothing: their rows of A are blanked
        if (t_begin + (long)TOK * (k + 1) > t_end) {
            for (int e = tid; e < TOK * 16; e += 256)
                if (t_begin + (long)TOK * k + e / 16 >= t_end) *(u32x4 *)(As + 8 * e) = u32x4{0u, 0u, 0u, 0u};
            __syncthreads();
        }
        multiply(As, As + TOK * 128);
    }
    products_done();
    float *out = J.Part + (size_t)share * J.KA * J.N;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int n = n0 + wn + 32 * y + c;
            if (n >= J.N) continue;
#pragma unroll
            for (int e = 0; e < 16; e += 4) {
                const int a = a0 + wa + 32 * x + 2 * e + 4 * h;
                if (a >= J.KA) continue;              // KA is a multiple of 8
#pragma unroll
                for (int d = 0; d < 4; ++d) out[(size_t)(a + d) * J.N + n] = acc[x][y][e + d];
            }
        }
}

__global__ __launch_bounds__(256, 2) void k_gemm_tn(GemmTn J0, GemmTn J1, long M, int share_tokens)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    tn_block(J0, J1, blockIdx.x, gridDim.x, M, share_tokens, (bf16_t *)lds);
}

// Out = In Wt^T and both contractions over the tokens in one launch: dX, dWqkv and dWo, once dQ, dK and dV are there.
// BM = 0: Out by split_tile.
template <int BM, int BN>
__global__ __launch_bounds__(256, 2) void k_gemm_bt_tn(GemmTn J0, GemmTn J1, int tiles, int share_tokens, const bf16_t *__restrict__ In,
                                                       const bf16_t *__restrict__ Wt, int ldw, int M, int K, int Nout, GemmOut out)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *lds = (bf16_t *)smem;
    if ((int)blockIdx.x < tiles) {
        if constexpr (BM == 0) split_tile<true, false, 4>(In, Wt, ldw, M, K, Nout, out, blockIdx.x, smem);
        else dma_tile<BM, BN, 2, true, false>(In, Wt, ldw, M, K, Nout, out, swizzled(blockIdx.x, tiles), lds);
        return;
    }
    tn_block(J0, J1, (int)blockIdx.x - tiles, (int)gridDim.x - tiles, M, share_tokens, lds);
}

template <int BM, int BN>
int launch_bt_tn(const GemmTn &J0, const GemmTn &J1, long tn_blocks, int share_tokens, const GemmHalf &b, long M, int K, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_gemm_bt_tn<BM, BN>, opted)) return BRA_ERR_LAUNCH;
    long blocks;
    size_t bytes;
    if constexpr (BM == 0) {
        blocks = split_blocks(M, b.Nout);
        bytes = split_bytes<4>();
    } else {
        blocks = tile_blocks<BM, BN>(M, b.Nout);
        bytes = ring_bytes<BM, BN, 2>();
    }
    if (tn_blocks + blocks > 0x7fffffffL) return BRA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((k_gemm_bt_tn<BM, BN>), dim3((unsigned)(tn_blocks + blocks)), dim3(256), std::max(kTnBytes, bytes), st,
                       J0, J1, (int)blocks, share_tokens, b.In, b.W, b.ldw, (int)M, K, b.Nout, b.out);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

bool sizes_ok(long M, int K, int Nout) { return M >= 1 && M <= 0x7fffffffL && K >= 64 && K % 64 == 0 && Nout >= 8 && Nout % 8 == 0; }

}  // namespace

int gemm(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out, const GemmRegions *regions,
         int kernel_id, hipStream_t st)
{
    if (!sizes_ok(M, K, Nout) || (out.cols % 32 && out.cols != Nout) || (out.in_rows.Hp && K > 4096)) return BRA_ERR_UNSUPPORTED;
    if (proj_ok(M, K, Nout, out, regions != nullptr)) {
        if (regions) {
            const int rc = gemm_regions(*regions, W, ldw, K, kernel_id, st);
            if (rc != BRA_OK) return rc;
        }
        ProfScope ps(st, kernel_id);
        return launch_proj(In, W, ldw, M, K, Nout, out, st);
    }
    ProfScope ps(st, kernel_id);
    // float32 copies: as with Q, K and V for all callers (bra_route decides on the same bits as bra_forward)
    if (!regions && splits(split_blocks(M, out.f32[0] ? 3 * out.cols : Nout), K, Nout, out.cols)) return launch_split(In, W, ldw, M, K, Nout, out, st);
    if (regions) return launch_big<true>(In, W, ldw, M, K, Nout, out, *regions, st);
    return launch_big<false>(In, W, ldw, M, K, Nout, out, GemmRegions{}, st);
}

int gemm_means(const bf16_t *In, const bf16_t *W, int ldw, int K, int Nout, const GemmOut &out, const GemmMeans &means, int kernel_id, hipStream_t st)
{
    const long M = (long)means.regions * means.n;
    if (!sizes_ok(M, K, Nout) || out.cols % 32 || K > 4096 || means.n > kMeansMaxTokens) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    // as with Q, K and V for both callers: bra_route decides on the same bits as bra_forward
    const long each = means.n <= 32 ? 32 / means.n : 0, rows = each ? (means.regions + each - 1) / each : 0;
    if (each && splits(rows * (3 * out.cols / 32), K, Nout, out.cols)) {
        static bool opted = false;
        if (!opt_in(k_gemm_means_split, opted)) return BRA_ERR_LAUNCH;
        hipLaunchKernelGGL(k_gemm_means_split, dim3((unsigned)(rows * (Nout / 32))), dim3(64 * kSplitWaves), split_bytes<kSplitWaves>(), st, In, W, ldw, K, Nout, out, means);
        return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
    }
    switch (pick_tile(M, K, Nout, 0, 0, means.n)) {
    case kOneChunk: return launch_means<64, 64, 1>(In, W, ldw, K, Nout, out, means, st);
    case kWide: return launch_means<128, 128, 2>(In, W, ldw, K, Nout, out, means, st);
    case kMid: return launch_means<64, 128, 2>(In, W, ldw, K, Nout, out, means, st);
    default: return launch_means<64, 64, 2>(In, W, ldw, K, Nout, out, means, st);
    }
}

int gemm_bt(const bf16_t *In, const bf16_t *Wt, int ldw, long M, int K, int Nout, bf16_t *Out, int kernel_id, hipStream_t st)
{
    if (!sizes_ok(M, K, Nout)) return BRA_ERR_UNSUPPORTED;
    const GemmOut out = {{Out, nullptr, nullptr}, Nout, {nullptr, nullptr}, nullptr, nullptr, 0};
    ProfScope ps(st, kernel_id);
    return launch_big<false, true>(In, Wt, ldw, M, K, Nout, out, GemmRegions{}, st);
}

int gemm_pair(const GemmHalf &a, const GemmHalf &b, long M, int K, int kernel_id, hipStream_t st)
{
    if (!sizes_ok(M, K, a.Nout) || !sizes_ok(M, K, b.Nout)) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    if (b.Nout == K && proj_ok(M, K, a.Nout, a.out, false) && a.Nout == 3 * K)
        return K == 64 ? launch_proj_t<64, 192, true>(a.In, a.W, a.ldw, M, a.out, st, b) : launch_proj_t<128, 384, true>(a.In, a.W, a.ldw, M, a.out, st, b);
    if (a.Nout % 32 == 0 && splits(split_blocks(M, a.Nout) + split_blocks(M, b.Nout), K, b.Nout, a.out.cols) && b.out.cols % 32 == 0) {
        static bool opted = false;
        if (!opt_in(k_gemm_pair_split, opted)) return BRA_ERR_LAUNCH;
        const long b0 = split_blocks(M, a.Nout), b1 = split_blocks(M, b.Nout);
        hipLaunchKernelGGL(k_gemm_pair_split, dim3((unsigned)(b0 + b1)), dim3(64 * kSplitWaves), split_bytes<kSplitWaves>(), st, a.In, a.W, a.ldw, a.Nout, a.out,
                           b.In, b.W, b.ldw, b.Nout, b.out, (int)M, K, (int)b0);
        return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
    }
    // tiles of both together
    switch (pick_tile(M, K, a.Nout, b.Nout, 0)) {
    case kOneChunk: return launch_pair<64, 64, 1>(a, b, M, K, st);
    case kWide: return launch_pair<128, 128, 2>(a, b, M, K, st);
    case kMid: return launch_pair<64, 128, 2>(a, b, M, K, st);
    default: return launch_pair<64, 64, 2>(a, b, M, K, st);
    }
}

// Shares of the tokens: at most two workgroups per compute unit over the 128 x 128 blocks of both products, and fewer where a
// share's partial matrices cost more to write and to add up again than its 64-token chunks cost to multiply: chunks / shares x
// 0.6 us + shares x elements x 1.8 ps is least at `paid`.  Whole gradient with 512 / blocks shares and now (us): 16 x 14 x 14 x 256,
// k = 16 59.2 / 56.1, 8 x 14 x 14 x 384 57.0 / 52.9, 16 x 7 x 7 x 512 64.4 / 59.4, 16 x 28 x 28 x 128, k = 4 60.2 / 55.6,
// 64 x 14 x 14 x 384 186.1 / 183.0; nearly as many shares as before, and nothing gained, 32 x 14 x 14 x 512 131.8 / 133.1.  One workgroup
// per compute unit throughout was faster yet at C = 128 (100 x 28 x 28, k = 4 209.7 to 212.8) and slower where shares are
// long: 16 x 14 x 14 x 1024 193 to 177.
static int tn_share_tokens(long M, int KA0, int N0, int KA1, int N1)
{
    auto blocks = [](int a, int n) { return (long)((a + 127) / 128) * ((n + 127) / 128); };
    const long chunks = (M + 63) / 64, paid = lrint(sqrt(3.3e5 * chunks / ((double)KA0 * N0 + (double)KA1 * N1)));
    const long want = std::max(1L, std::min(512 / (blocks(KA0, N0) + blocks(KA1, N1)), paid));
    return (int)((chunks + want - 1) / want * 64);
}

// Workgroups of both products, a multiple of 8.
static long tn_blocks(const GemmTn &J0, const GemmTn &J1, int shares)
{
    auto blocks = [](const GemmTn &J) { return (long)((J.KA + 127) / 128) * ((J.N + 127) / 128); };
    return ((blocks(J0) + blocks(J1)) * shares + 7) / 8 * 8;
}

int gemm_tn_shares(long M, int KA0, int N0, int KA1, int N1)
{
    const int t = tn_share_tokens(M, KA0, N0, KA1, N1);
    return (int)((M + t - 1) / t);
}

int gemm_tn(const GemmTn &J0, const GemmTn &J1, long M, int kernel_id, hipStream_t st)
{
    if (M < 1 || (J0.KA | J0.N | J1.KA | J1.N | J0.lda | J0.ldb | J1.lda | J1.ldb) % 8) return BRA_ERR_UNSUPPORTED;
    const int tokens = tn_share_tokens(M, J0.KA, J0.N, J1.KA, J1.N), shares = gemm_tn_shares(M, J0.KA, J0.N, J1.KA, J1.N);
    static bool opted = false;
    if (!opt_in(k_gemm_tn, opted)) return BRA_ERR_LAUNCH;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL(k_gemm_tn, dim3((unsigned)tn_blocks(J0, J1, shares)), dim3(256), kTnBytes, st, J0, J1, M, tokens);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

// One launch where the product by itself leaves the chip under-filled, up to 256 tiles of 128 x 128.  Whole gradient with two
// launches and one (us): 8 x 14 x 14 x 256, k = 16 (26 tiles) 47.7 / 43.1; 2 x 7 x 7 x 768 (6) 57.0 / 50.5; 16 x 7 x 7 x 512 (28)
// 64 / 59; above, each fills the chip and the two get into each other's way: 64 x 14 x 14 x 384 (294) 181 / 184, 8 x 32 x 32 x 768
// (384) 258 / 266.
int gemm_bt_tn(const GemmTn &J0, const GemmTn &J1, const GemmHalf &b, long M, int K, int kernel_id, hipStream_t st)
{
    if (tile_blocks<128, 128>(M, b.Nout) > 256) {
        const int rc = gemm_bt(b.In, b.W, b.ldw, M, K, b.Nout, (bf16_t *)b.out.buf[0], kernel_id, st);
        return rc == BRA_OK ? gemm_tn(J0, J1, M, kernel_id, st) : rc;
    }
    if (!sizes_ok(M, K, b.Nout) || (J0.KA | J0.N | J1.KA | J1.N | J0.lda | J0.ldb | J1.lda | J1.ldb) % 8) return BRA_ERR_UNSUPPORTED;
    const int tokens = tn_share_tokens(M, J0.KA, J0.N, J1.KA, J1.N), shares = gemm_tn_shares(M, J0.KA, J0.N, J1.KA, J1.N);
    const long tn = tn_blocks(J0, J1, shares);
    ProfScope ps(st, kernel_id);
    // beside the contractions, with four wavefronts, up to half as many tiles unless the walk is long; then up to as many as it has steps of 16, or 112. Tiles, whole call with
    // tiles of 64 / split (us): K = 768 (28) 29.1 / 28.0; K = 576 (48) 31.1 / 32.5; K = 1152 (60) 46.3 / 45.8, (72) 36.2 / 35.6 and 47.4 / 47.6, (96) 37.1 / 37.7, (114) 44.4 / 48.3;
    // K = 1536 (96) 52.0 / 50.6, (104) 41.2 / 42.7, (112) 64.3 / 66.7; K = 2304 (84) 49.5 / 44.2, (108) 73.1 / 72.8, (120) 73.7 / 74.5.
    if (splits(split_blocks(M, b.Nout), K, b.Nout, b.out.cols) && (M + 63) / 64 * ((b.Nout + 63) / 64) <= (K >= 1024 ? std::min(K / 16, 112) : 32)) return launch_bt_tn<0, 0>(J0, J1, tn, tokens, b, M, K, st);
    // that few tiles are never the wide ones
    if (pick_tile(M, K, b.Nout, 0, 0) == kNarrow) return launch_bt_tn<64, 64>(J0, J1, tn, tokens, b, M, K, st);
    return launch_bt_tn<64, 128>(J0, J1, tn, tokens, b, M, K, st);
}

int gemm_regions(const GemmRegions &r, const bf16_t *W, int ldw, int K, int kernel_id, hipStream_t st)
{
    if (!sizes_ok(r.M, K, r.Nout)) return BRA_ERR_UNSUPPORTED;
    ProfScope ps(st, kernel_id);
    // 64 x 64 tiles (twice the workgroups, six wavefronts per SIMD instead of four) where 64 x 128
    // tiles would leave the chip under-filled; measured: the narrow tile wins below a few hundred
    // wide tiles and loses above about a thousand
    // (and where the output is at most 64 columns wide: half of a wide tile would be idle)
    const long mt = (r.M + 63) / 64;
    if (r.Nout <= 64 || mt * ((r.Nout + 127) / 128) < 400)
        hipLaunchKernelGGL(k_gemm<2>, dim3((unsigned)(mt * ((r.Nout + 63) / 64))), dim3(256), 0, st, r, W, ldw, K);
    else
        hipLaunchKernelGGL(k_gemm<4>, dim3((unsigned)(mt * ((r.Nout + 127) / 128))), dim3(256), 0, st, r, W, ldw, K);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

int gemm_bf16(const bf16_t *In, const bf16_t *W, long M, int K, int Nout, bf16_t *Out, const float *bias,
              const bf16_t *res, bool gelu, int kernel_id, hipStream_t st)
{
    return gemm(In, W, Nout, M, K, Nout, GemmOut{{Out, nullptr, nullptr}, Nout, {nullptr, nullptr}, bias, res, gelu ? 1 : 0},
                nullptr, kernel_id, st);
}

}  // namespace bra
