// Attention backward for regions of any size (bf16, heads of 32 or 64 channels, C a multiple of 64): two kernels with the
// layout of the forward's k_attn_gen and k_attn_rows (bra_mfma_wide.hip).
//
// With P = 2^(S - lse), S = Q K^T in units of log2 (Q comes multiplied by scale log2(e)), the row statistics enter the
// products as their accumulator inputs: S - lse and dP - D, D = rowsum(dO o O), leave the matrix cores ready for
//     dS = 2^(S - lse) (dP - D)                        an exponential, a multiplication and half a conversion per score
// with dP = dO V^T, dQ = scale dS K, dV = P^T dO, dK = scale dS^T Q.
//
// kShared: a workgroup takes 64 N tokens of one region (16 N per wavefront) and 64 channels (2 or 1 heads); blocks of 64
// rows of the other side are shared by its wavefronts.  kWaves (regions of at most 32 tokens): a wavefront takes all
// tokens of a region and 64 channels by itself, with blocks of 32 rows in its own part of LDS and no barriers.  kSplit
// (small calls): the wavefronts of a workgroup take every fourth block for the same 16 N tokens and add up at the end.  Rows
// (128 bytes of each of two maps) go straight from memory into one of two buffers while the other is worked on; their
// 16-byte pieces are exchanged (piece c of row r at c ^ r % 8), so that row reads and transposing reads meet different banks.
//
// Measured, query side + key side (us; before: kernels that staged rows through registers and formed S and dP without
// their statistics): 11 x 42 x 42 x 256, k = 6 (36 tokens per region): 77 + 66 -> 54 + 44; 25 x 8 x 16 x 768 with heads
// of 64, k = 36 (2 tokens): 215 + 172 -> 65 + 88; 12 x 112 x 120 x 64, k = 1 (210 tokens): 112 + 105 -> 68 + 75;
// 64 x 56 x 56 x 64, k = 1: 36 + 49 -> 39 + 41, there bound by memory (150 MB per kernel).  D = dO . O instead of the sum
// over the keys took 47, 65, 68 and 37 us on the query side, with the rounding of the bf16 weights in D.
//
// Both launches also carry a pass of the depth-wise convolution's gradients (bra_lce_pairs.h), which needs nothing of them: the
// query side LCE^T(dO) in float32 with the tap gradients, the key side O += LCE(V), and adds its dV to what is there (rounded to bf16
// there, LCE^T(dO) put 4 to 6 % on the error of dX from float64; now 0.5 % below that of a convolution added to a rounded dV).
// Each launch costs about 6 us to fill and to drain the chip, and neither kind of work alone keeps the memory busy.  Whole
// gradient with launches of their own and here (us): 1 x 56 x 56 x 64, k = 1: 39.2 -> 31.7; 16 images: 87.6 -> 77.9;
// 64 x 28 x 28 x 128, k = 4: 144 -> 140; 8 x 56 x 56 x 256, k = 4: 200 -> 186; 12 x 112 x 120 x 64: 251 -> 237.  Large maps: BackwardJobs.
//
// LCE: where a workgroup has its region whole and all routed keys in one block, the query side adds LCE(V) to O and the key side begins dV with
// LCE^T(dO), both from the region's halo in LDS (bra_lce_region.h): 26 bytes per value less to move (the float32 between the
// two kernels, O read and written once more, V and dO read once more), and O is rounded once (error of dWo of 64 x 56 x 56 x 64 from
// float64 2.44e-3 -> 2.26e-3).  The tap gradients alone stay a pass.  Together with SINGLE, 64 x 56 x 56 x 64, k = 1: query side 71 -> 55 us,
// key side 66 -> 58, whole gradient 209 -> 181; 16 images 79.3 -> 77.9, 2 images 40.0 -> 40.1.  Of the key side's 58 us the attention takes 43, the
// products of the convolution 6, the halo's loads 5; the list of regions made while they arrive gave nothing, and the convolution
// beside the first block costs 90 registers of scratch.  Four
// wavefronts per SIMD spill 6 registers of the key side; three, which spill none: 64 x 56 x 56 x 64 178.8 -> 180.5 us, 16 images 74.2 -> 74.5.  With more than one block (36 tokens, k = 6; 63 tokens, k = 4) it is 0 to 9 % slower than the passes.
// SINGLE: all routed keys in one block: a head's scores and dP stay in registers from the weights to dS, which takes out the second sweep (a
// third of the vector instructions) and 50 registers; 44 x 21 x 21 x 512, k = 2 281 -> 275 us.
#include "bra_attn_dev.h"
#include "bra_lce_region.h"
#include "bra_mfma_bwd_attn.h"

namespace bra {

using namespace mfma;

namespace {

enum Mode { kWaves, kShared, kSplit };

template <Mode MODE>
struct Rows {
    static constexpr bool SHARED = MODE == kShared;
    static constexpr int KB = SHARED ? 64 : 32;                // rows of a block
    static constexpr int per_wave = SHARED ? 16 : 32;          // rows that a wavefront brings
    static constexpr int buf = 2 * KB * 64;                    // elements of a buffer: two maps
    static constexpr int bufs = 2 * (SHARED ? 1 : 4);          // two per workgroup or wavefront
};

// The workgroup's or wavefront's place in the grid: (image, region, tile of tokens, group of 64 channels); false: none.
template <Mode MODE>
__device__ __forceinline__ bool place(const Dims &D, int tiles, int items, int wid, int wave, int &b, int &reg, int &tile, int &cg)
{
    const int ncg = D.C / 64;
    const int item = MODE != kWaves ? wid : __builtin_amdgcn_readfirstlane(4 * wid + wave);
    if (item >= items) return false;
    cg = item % ncg;
    tile = (item / ncg) % tiles;
    reg = (item / (ncg * tiles)) % D.R;
    b = item / (ncg * tiles * D.R);
    return true;
}

// Items of a lane group at most (lce::halo_sums).
constexpr int kLceRounds = 2;

// ---------------------------------------------------------------------------
// Query side: attention output O, row statistics lse and D, and dQ, in two sweeps over the region's k n routed keys.  The
// first is the forward's attention and sums D = sum P dP beside it, from the float32 weights (dO . O has the rounding of
// the weights that entered O).  The second goes over the blocks backwards, so that the
// last two are still in LDS (up to 128 or 64 routed keys: nothing is read twice).
template <int HD, int NQ, Mode MODE, bool LCE, bool SINGLE>
__global__ __launch_bounds__(256, MODE == kShared && NQ == 1 ? (LCE ? 4 : 3) : 2) void k_attn_bwd_q(AttnBwdArgs A, Dims D, int tiles, int items, int walks, lce::Job J,
                                                                                                     int lce_blocks, int lce_front)
{
    using R = Rows<MODE>;
    constexpr bool SHARED = R::SHARED, SPLIT = MODE == kSplit;
    constexpr int HPW = 64 / HD, KSD = HD / 32, NDT = HD / 16, KB = R::KB, KT = KB / 16;
    static_assert(!LCE || (SINGLE && SHARED && NQ == 1), "one block, one tile");
    __shared__ __attribute__((aligned(16))) bf16_t lds[LCE ? R::buf : R::bufs * R::buf];
    constexpr int kPart = 64 * (3 + 4 * NDT);    // SPLIT: m, l, D and the sums of a wavefront, one query tile and head
    __shared__ __attribute__((aligned(16))) float sums[SPLIT ? NQ * HPW * 4 * kPart : 4];
    static_assert((LCE ? lce::kTapSumBytes : lce::job_bytes<true>()) <= sizeof(lds), "the pass shares the buffers");
    // LCE: the halo of V, then LCE(V) of the tokens; [k] or [4][k]: first token of the routed regions; with `walks` [n] or [4][n]: tokens of a region's slots
    extern __shared__ __attribute__((aligned(16))) int origin_tables[];
    int wg, wgs;
    if (lce::block_of_pass(lce_blocks, lce_front, wg, wgs)) {
        if constexpr (LCE) lce::taps_block(J, D, swizzled(wg, wgs), (float *)lds);
        else lce::job_block<true, false>(J, D, swizzled(wg, wgs), (float *)lds);
        return;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int C = D.C, n = D.n, kn = D.kn;
    int b, reg, tile, cg;
    if (!place<MODE>(D, tiles, items, swizzled(wg, wgs), wave, b, reg, tile, cg)) return;
    const Places<false> at(D);
    const float n_inv = 1.0f / (float)n;
    const size_t img = (size_t)b * D.N * C + 64 * cg;
    bf16_t *mine = lds + (SHARED ? 0 : wave * 2 * R::buf);
    const lce::RegionHalo halo(D.rh, D.rw);
    int *const tables = origin_tables + (LCE ? halo.bytes(n) / 4 : 0);
    const lce::LaneTaps<false> taps(J.Wlce, 64 * cg + (LCE ? 16 * wave + lane % 16 : 0));
    int *origins = tables + (SHARED ? 0 : wave * D.k), *slots = tables + (SHARED ? D.k : 4 * D.k + wave * n);
    if (LCE || walks)
        for (int t = SHARED ? tid : lane; t < n; t += SHARED ? 256 : kWave) slots[t] = at.slot(t);
    for (int p = SHARED ? tid : lane; p < D.k; p += SHARED ? 256 : kWave)
        origins[p] = at.origin(region_index(A.Ir[((size_t)b * D.R + reg) * D.k + p], D.R));
    const int q0 = SHARED ? 64 * NQ * tile + 16 * NQ * wave : 16 * NQ * tile;
    const bool idle = SHARED && q0 >= n;         // a wavefront without queries only brings its rows
    int tok[NQ];
    bf16x8 qf[NQ][HPW][KSD], gf[NQ][HPW][KSD];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        tok[q] = at.origin(reg) + at.slot(min(q0 + 16 * q + i, n - 1));
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) {
                const size_t e = img + (size_t)tok[q] * C + HD * hh + 32 * ks + 8 * g;
                qf[q][hh][ks] = *(const bf16x8 *)(A.Q + e);
                gf[q][hh][ks] = *(const bf16x8 *)(A.dO + e);
            }
    }
    // the operands have arrived before the sweeps: otherwise the compiler waits for them there, and with them for the
    // direct loads in flight
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) asm volatile("" : "+v"(qf[q][hh][ks]), "+v"(gf[q][hh][ks]));
    unsigned w[5][3];
    if constexpr (LCE) {
        taps.operands(w);
#pragma unroll
        for (int ky = 0; ky < 5; ++ky) asm volatile("" : "+v"(w[ky][0]), "+v"(w[ky][1]), "+v"(w[ky][2]));
    }
    if (SHARED) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the table is read by other lanes

    // blocks of this wavefront: local block s is block STEP s + start
    constexpr int STEP = SPLIT ? 4 : 1;
    const int start = SPLIT ? wave : 0, nb = ((kn + KB - 1) / KB - start + STEP - 1) / STEP;
    // The walk stands at the block to be requested next: upwards in the first sweep, back in the second.
    constexpr int LOADS = R::per_wave / 8;
    RowWalk<LOADS> walk;
    walk.start(KB * start + (SHARED ? 16 * wave : 0) + lane / 8, 8, KB * STEP, n, n_inv);
    const unsigned piece = 16 * ((lane % 8) ^ (lane / 8)), my_lds = lds_address(mine) + (SHARED ? 2048 * wave : 0);
    auto request = [&](int local, bool back) {
        const unsigned to = my_lds + (local % 2) * (2 * R::buf);
        lds_reads_done();
        if (back) walk.retreat();
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            if (MODE == kWaves || LCE || walks) {
                const unsigned off = row_offset(walk.token(u, origins, D.k - 1, slots), C, piece);
                load_to_lds_untracked(A.K + img, off, to + 1024 * u);
                load_to_lds_untracked(A.V + img, off, to + KB * 128 + 1024 * u);
            } else {
                const int row = (SHARED ? 16 * wave : 0) + 8 * u + lane / 8, key = min(KB * (STEP * local + start) + row, kn - 1), p = divide(key, n, n_inv);
                const size_t e = img + (size_t)(origins[p] + at.slot(key - p * n)) * C + piece / 2;
                load_to_lds_untracked(A.K + e, to + 1024 * u);
                load_to_lds_untracked(A.V + e, to + KB * 128 + 1024 * u);
            }
        }
        if (!back) walk.advance();
    };
    // Step s works on block s of the first sweep, then backwards; the first two blocks of the second sweep are in place.
    // On return the block of step s is in LDS and that of step s + 1 requested.
    auto block_of = [&](int s) { return s < nb ? s : 2 * nb - 1 - s; };
    auto advance = [&](int s) {
        const bool more = !SINGLE && s + 1 < 2 * nb && (s + 1 < nb || s + 1 > nb + 1);
        if (s + 1 == nb + 2) {                   // from behind the last block to the one before the two that are in place
            walk.retreat();
            walk.retreat();
        }
        if (SHARED) {
            arrive_barrier();
            if (more) request(block_of(s + 1), s >= nb);
        } else if (more) {
            request(block_of(s + 1), s >= nb);
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    };
    float m[NQ][HPW], l[NQ][HPW], dd[NQ][HPW];
    f32x4 acc[NQ][HPW][NDT];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            m[q][hh] = l[q][hh] = dd[q][hh] = 0.f;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) acc[q][hh][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto mask = [&](f32x4 (&s)[KT], int left) {              // keys past the end get no weight
        if (left < KB) {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (16 * t + 4 * g + j >= left) s[t][j] = -INFINITY;
        }
    };
    auto forward = [&](int s, auto first) {
        const bf16_t *Ks = mine + (s % 2) * R::buf, *Vs = Ks + KB * 64;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            bf16x8 pb[NQ][KT / 2];
            {
                bf16x8 kf[KT][KSD], vr[KT][KSD];
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int ks = 0; ks < KSD; ++ks) {
                        kf[t][ks] = row_operand(Ks, 16 * t + i, HD / 8 * hh + 4 * ks + g);
                        vr[t][ks] = row_operand(Vs, 16 * t + i, HD / 8 * hh + 4 * ks + g);
                    }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    f32x4 sc[KT], dp[KT];
                    const float neg = -m[q][hh];
#pragma unroll
                    for (int t = 0; t < KT; ++t) {
                        sc[t] = f32x4{neg, neg, neg, neg};
                        dp[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int ks = 0; ks < KSD; ++ks) {
                            sc[t] = mfma16(kf[t][ks], qf[q][hh][ks], sc[t]);   // S^T[key 16 t + 4 g + j][query i]
                            dp[t] = mfma16(vr[t][ks], gf[q][hh][ks], dp[t]);
                        }
                    }
                    mask(sc, kn - KB * (STEP * s + start));
                    softmax_step<decltype(first)::value>(sc, m[q][hh], l[q][hh], acc[q][hh], pb[q], dp, &dd[q][hh]);
                    if (SHARED && NQ > 1) __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int tp = 0; tp < KT / 2; ++tp)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const bf16x8 vf = column_operand(Vs, 32 * tp, HD * hh + 16 * dt, g, i);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) acc[q][hh][dt] = mfma16(vf, pb[q][tp], acc[q][hh][dt]);
                }
            if (SHARED) __builtin_amdgcn_sched_barrier(0);    // one head at a time: interleaved, they take twice the registers
        }
    };
    if (!SPLIT || nb > 0) {
        if constexpr (LCE) {
            const int ry = fast_div(reg, at.s_inv);
            lce::request_halo(halo, A.V + img, D, ry * D.rh, (reg - ry * D.S) * D.rw, lds_address(origin_tables), wave, lane);
        }
        request(0, false);
        if constexpr (LCE) {
            asm volatile("s_waitcnt vmcnt(%0)" : : "i"(2 * LOADS) : "memory");       // the halo is there, the block need not be
            __syncthreads();
            float o[kLceRounds][4][4];
            lce::halo_sums<kLceRounds>(halo, (const bf16_t *)origin_tables, w, wave, lane, o);
            __syncthreads();                     // the halo has been read
            lce::park_sums<kLceRounds>(halo, D, (float *)origin_tables, wave, lane, o);
        }
        advance(0);
        if constexpr (!SINGLE) {
            if (!idle) forward(0, std::true_type{});
        }
    }
    if constexpr (SINGLE) {
        // a head at a time, its scores and dP in registers from beginning to end
        if (idle) return;
        const bf16_t *Ks = mine, *Vs = Ks + KB * 64;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            f32x4 sc[NQ][KT], dp[NQ][KT];
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                bf16x8 kf[KSD], vf[KSD];
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    kf[ks] = row_operand(Ks, 16 * t + i, HD / 8 * hh + 4 * ks + g);
                    vf[ks] = row_operand(Vs, 16 * t + i, HD / 8 * hh + 4 * ks + g);
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    sc[q][t] = dp[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KSD; ++ks) {
                        sc[q][t] = mfma16(kf[ks], qf[q][hh][ks], sc[q][t]);       // S^T[key 16 t + 4 g + j][query i]
                        dp[q][t] = mfma16(vf[ks], gf[q][hh][ks], dp[q][t]);
                    }
                }
            }
            bf16x8 pb[NQ][KT / 2], db[NQ][KT / 2];
            float inv[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                mask(sc[q], kn);
                float mx = sc[q][0][0];
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) mx = fmaxf(mx, sc[q][t][j]);
                mx = cross_row_max(mx);
                float sum = 0.f, d = 0.f;
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        sc[q][t][j] = __builtin_amdgcn_exp2f(sc[q][t][j] - mx);
                        sum += sc[q][t][j];
                        d = fmaf(sc[q][t][j], dp[q][t][j], d);
                    }
                sum = cross_row_sum(sum);
                inv[q] = 1.0f / sum;
                d = cross_row_sum(d) * inv[q];
#pragma unroll
                for (int tp = 0; tp < KT / 2; ++tp) {
                    float p[8], ds[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        p[e] = sc[q][2 * tp + e / 4][e % 4];
                        ds[e] = p[e] * inv[q] * (dp[q][2 * tp + e / 4][e % 4] - d);
                    }
                    pb[q][tp] = pack8(p);
                    db[q][tp] = pack8(ds);
                }
                if (q0 + 16 * q + i < n && g == 0) {
                    const size_t e = ((size_t)b * D.heads + HPW * cg + hh) * D.N + tok[q];
                    A.lse[e] = mx + __builtin_amdgcn_logf(sum);                  // v_log_f32: log2
                    A.dsum[e] = d;
                }
            }
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                f32x4 o[NQ], dq[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) o[q] = dq[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int tp = 0; tp < KT / 2; ++tp) {
                    const bf16x8 vc = column_operand(Vs, 32 * tp, HD * hh + 16 * dt, g, i), kc = column_operand(Ks, 32 * tp, HD * hh + 16 * dt, g, i);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        o[q] = mfma16(vc, pb[q][tp], o[q]);
                        dq[q] = mfma16(kc, db[q][tp], dq[q]);
                    }
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int slot = q0 + 16 * q + i;
                    if (slot >= n) continue;
                    const int ch = HD * hh + 16 * dt + 4 * g;
                    f32x4 v = o[q] * inv[q];
                    if constexpr (LCE) v += *(const f32x4 *)((const float *)origin_tables + slot * lce::kResultPitch + ch);
                    *(u32x2 *)(A.O + img + (size_t)tok[q] * C + ch) = pack4(v);
                    *(u32x2 *)(A.dQKV + ((size_t)b * D.N + tok[q]) * 3 * C + 64 * cg + ch) = pack4(dq[q] * D.scale);
                }
            }
            if (SHARED) __builtin_amdgcn_sched_barrier(0);    // one head at a time: interleaved, they take twice the registers
        }
        return;
    }
#pragma unroll 1
    for (int s = 1; s < nb; ++s) {
        advance(s);
        if (!idle) forward(s, std::false_type{});
    }
    if constexpr (SPLIT) {
        // the four wavefronts' sums on a common reference
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                if (nb == 0) m[q][hh] = -INFINITY;
                float *part = sums + (q * HPW + hh) * 4 * kPart + lane;
                part[wave * kPart] = m[q][hh];
                part[wave * kPart + 64] = l[q][hh];
                part[wave * kPart + 128] = dd[q][hh];
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int j = 0; j < 4; ++j) part[wave * kPart + 64 * (3 + 4 * dt + j)] = acc[q][hh][dt][j];
            }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                const float *part = sums + (q * HPW + hh) * 4 * kPart + lane;
                const float top = fmaxf(fmaxf(part[0], part[kPart]), fmaxf(part[2 * kPart], part[3 * kPart]));
                float f[4], sum = 0.f, dsum = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    f[w] = __builtin_amdgcn_exp2f(part[w * kPart] - top);
                    sum += f[w] * part[w * kPart + 64];
                    dsum += f[w] * part[w * kPart + 128];
                }
                m[q][hh] = top;
                l[q][hh] = sum;
                dd[q][hh] = dsum;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float a = 0.f;
#pragma unroll
                        for (int w = 0; w < 4; ++w) a += f[w] * part[w * kPart + 64 * (3 + 4 * dt + j)];
                        acc[q][hh][dt][j] = a;
                    }
            }
    }
    float neg_lse[NQ][HPW], neg_d[NQ][HPW];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const bool store = q0 + 16 * q + i < n && (!SPLIT || wave == 0);
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            const float total = cross_row_sum(l[q][hh]), inv = 1.0f / total, d = cross_row_sum(dd[q][hh]) * inv;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                if (store) *(u32x2 *)(A.O + img + (size_t)tok[q] * C + HD * hh + 16 * dt + 4 * g) = pack4(acc[q][hh][dt] * inv);
                acc[q][hh][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            const float lse = m[q][hh] + __builtin_amdgcn_logf(total);       // v_log_f32: log2
            neg_lse[q][hh] = -lse;
            neg_d[q][hh] = -d;
            if (store && g == 0) {
                const size_t e = ((size_t)b * D.heads + HPW * cg + hh) * D.N + tok[q];
                A.lse[e] = lse;
                A.dsum[e] = d;
            }
        }
    }
#pragma unroll 1
    for (int s = nb; s < 2 * nb; ++s) {
        advance(s);
        if (idle) continue;
        const int local = block_of(s), blk = STEP * local + start;
        const bf16_t *Ks = mine + (local % 2) * R::buf, *Vs = Ks + KB * 64;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh) {
            bf16x8 db[NQ][KT / 2];
#pragma unroll
            for (int tp = 0; tp < KT / 2; ++tp) {
                f32x4 sc[NQ][2], dp[NQ][2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    bf16x8 kf[KSD], vf[KSD];
#pragma unroll
                    for (int ks = 0; ks < KSD; ++ks) {
                        kf[ks] = row_operand(Ks, 32 * tp + 16 * t + i, HD / 8 * hh + 4 * ks + g);
                        vf[ks] = row_operand(Vs, 32 * tp + 16 * t + i, HD / 8 * hh + 4 * ks + g);
                    }
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const float a = neg_lse[q][hh], c = neg_d[q][hh];
                        sc[q][t] = f32x4{a, a, a, a};
                        dp[q][t] = f32x4{c, c, c, c};
#pragma unroll
                        for (int ks = 0; ks < KSD; ++ks) {
                            sc[q][t] = mfma16(kf[ks], qf[q][hh][ks], sc[q][t]);
                            dp[q][t] = mfma16(vf[ks], gf[q][hh][ks], dp[q][t]);
                        }
                    }
                }
                const int left = kn - KB * blk - 32 * tp;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    if (left < 32) {
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                if (16 * t + 4 * g + j >= left) sc[q][t][j] = -INFINITY;
                    }
                    float ds[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) ds[e] = __builtin_amdgcn_exp2f(sc[q][e / 4][e % 4]) * dp[q][e / 4][e % 4];
                    db[q][tp] = pack8(ds);
                }
            }
#pragma unroll
            for (int tp = 0; tp < KT / 2; ++tp)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const bf16x8 kc = column_operand(Ks, 32 * tp, HD * hh + 16 * dt, g, i);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) acc[q][hh][dt] = mfma16(kc, db[q][tp], acc[q][hh][dt]);
                }
            if (SHARED) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (SPLIT) {
        // wavefront w adds up and stores channels 16 w .. 16 w + 15
        __syncthreads();                          // the sums have been read
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int a = 0; a < 4; ++a) *(f32x4 *)(sums + ((q * 4 + a) * 4 + wave) * 256 + 4 * lane) = acc[q][a / NDT][a % NDT];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (q0 + 16 * q + i >= n) continue;
            const float *part = sums + (q * 4 + wave) * 1024 + 4 * lane;
            const f32x4 sum = (*(const f32x4 *)part + *(const f32x4 *)(part + 256)) + (*(const f32x4 *)(part + 512) + *(const f32x4 *)(part + 768));
            *(u32x2 *)(A.dQKV + ((size_t)b * D.N + tok[q]) * 3 * C + 64 * cg + 16 * wave + 4 * g) = pack4(sum * D.scale);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q0 + 16 * q + i >= n) continue;
        bf16_t *row = A.dQKV + ((size_t)b * D.N + tok[q]) * 3 * C + 64 * cg + 4 * g;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) *(u32x2 *)(row + HD * hh + 16 * dt) = pack4(acc[q][hh][dt] * D.scale);
    }
}

// ---------------------------------------------------------------------------
// Key side: dK and dV of a region's tokens, summed in registers over the queries of all regions routed to it (every entry
// of Ir that names it, in the order of the entries, so the result is the same every time).
constexpr float kLn2 = 0.6931471805599453f;             // dK = scale dS^T Q, and Q came with scale log2(e)
constexpr int kListShared = 1024, kListWave = 512;      // entries listed at a time

// Query regions whose entries e0, e0 + 1, .. name region j, as first tokens, up to a full list; e0 moves behind the
// entries looked at.  A wavefront on its own.
__device__ __forceinline__ int list_of_wave(const int32_t *__restrict__ irb, int entries, int &e0, int j, int R, float k_inv,
                                            const Places<false> &at, int *list)
{
    const int lane = threadIdx.x % kWave;
    int count = 0;
    for (; e0 < entries && count + 4 * kWave <= kListWave; e0 += 4 * kWave) {
        int r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = irb[min(e0 + kWave * u + lane, entries - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + kWave * u + lane;
            const bool named = e < entries && region_index(r[u], R) == j;
            const unsigned long long votes = __ballot(named);
            if (named) list[count + __popcll(votes & ((1ull << lane) - 1))] = at.origin(fast_div(e, k_inv));
            count += __popcll(votes);
        }
    }
    return count;
}

// The same for the whole workgroup, one range of kListShared entries at a time; barriers around it are the caller's.
__device__ __forceinline__ int list_of_group(const int32_t *__restrict__ irb, int entries, int e0, int j, int R, float k_inv,
                                             const Places<false> &at, int *list, int *counts)
{
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    unsigned long long votes[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = e0 + 256 * u + (int)threadIdx.x;
        votes[u] = __ballot(e < entries && region_index(irb[min(e, entries - 1)], R) == j);
        if (lane == 0) counts[4 * u + wave] = __popcll(votes[u]);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == wave && (votes[u] >> lane & 1))
                list[total + __popcll(votes[u] & ((1ull << lane) - 1))] = at.origin(fast_div(e0 + 256 * u + (int)threadIdx.x, k_inv));
            total += counts[4 * u + w];
        }
    return __builtin_amdgcn_readfirstlane(total);
}

template <int HD, int NK, Mode MODE, bool LCE>
__global__ __launch_bounds__(256, MODE == kShared && NK == 1 ? (LCE ? 4 : 3) : 2) void k_attn_bwd_kv(AttnBwdArgs A, Dims D, int tiles, int items, int walks, lce::Job J, int lce_blocks)
{
    using R = Rows<MODE>;
    constexpr bool SHARED = R::SHARED, SPLIT = MODE == kSplit;
    constexpr int HPW = 64 / HD, KSD = HD / 32, NDT = HD / 16, KB = R::KB;
    constexpr int kStats = HPW * 2 * KB;         // per buffer: [head][lse, D][row]
    __shared__ __attribute__((aligned(16))) bf16_t lds[R::bufs * R::buf];
    __shared__ __attribute__((aligned(16))) float stats[R::bufs * kStats];
    __shared__ __attribute__((aligned(16))) float sums[SPLIT ? NK * 4 * 2048 : 4];
    __shared__ int lists[SHARED ? kListShared : 4 * kListWave];
    __shared__ int counts[16];
    int wg = blockIdx.x, wgs = gridDim.x;
    if (!LCE && lce::block_of_pass(lce_blocks, false, wg, wgs)) {
        lce::job_block<false, true>(J, D, swizzled(wg, wgs), (float *)lds);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) int slot_tables[];         // with `walks` [n] or [4][n]: tokens of a region's slots
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave, g = lane / 16, i = lane % 16;
    const int C = D.C, n = D.n;
    int b, reg, tile, cg;
    if (!place<MODE>(D, tiles, items, swizzled(wg, wgs), wave, b, reg, tile, cg)) return;
    const Places<false> at(D);
    const float n_inv = 1.0f / (float)n, k_inv = 1.0f / (float)D.k;
    const size_t img = (size_t)b * D.N * C + 64 * cg;
    const size_t stat0 = ((size_t)b * D.heads + HPW * cg) * D.N;
    bf16_t *mine = lds + (SHARED ? 0 : wave * 2 * R::buf);
    float *my_stats = stats + (SHARED ? 0 : wave * 2 * kStats);
    int *list = lists + (SHARED ? 0 : wave * kListWave), *slots = slot_tables + (SHARED ? 0 : wave * n);
    if (LCE || walks)
        for (int t = SHARED ? tid : lane; t < n; t += SHARED ? 256 : kWave) slots[t] = at.slot(t);

    const int q0 = SHARED ? 64 * NK * tile + 16 * NK * wave : 16 * NK * tile;
    const bool idle = SHARED && q0 >= n;         // a wavefront without keys only brings its rows
    int tok[NK];
    bf16x8 kf[NK][HPW][KSD], vf[NK][HPW][KSD];
#pragma unroll
    for (int q = 0; q < NK; ++q) {
        tok[q] = at.origin(reg) + at.slot(min(q0 + 16 * q + i, n - 1));
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) {
                const size_t e = img + (size_t)tok[q] * C + HD * hh + 32 * ks + 8 * g;
                kf[q][hh][ks] = *(const bf16x8 *)(A.K + e);
                vf[q][hh][ks] = *(const bf16x8 *)(A.V + e);
            }
    }
    f32x4 dk[NK][HPW][NDT], dv[NK][HPW][NDT];
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) dk[q][hh][dt] = dv[q][hh][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // dV begins with LCE^T(dO)
    if constexpr (LCE) {
        unsigned w[5][3];
        const lce::RegionHalo halo(D.rh, D.rw);
        const lce::LaneTaps<true> taps(J.Wlce, 64 * cg + 16 * wave + lane % 16);
        const int ry = fast_div(reg, at.s_inv);
        lce::request_halo(halo, A.dO + img, D, ry * D.rh, (reg - ry * D.S) * D.rw, lds_address(lds), wave, lane);
        taps.operands(w);
        arrive_barrier();
        float o[kLceRounds][4][4];
        lce::halo_sums<kLceRounds>(halo, lds, w, wave, lane, o);
        __syncthreads();                         // the halo has been read
        lce::park_sums<kLceRounds>(halo, D, (float *)lds, wave, lane, o);
        __syncthreads();
#pragma unroll
        for (int a = 0; a < HPW * NDT; ++a) dv[0][a / NDT][a % NDT] = *(const f32x4 *)((const float *)lds + min(q0 + i, n - 1) * lce::kResultPitch + 16 * a + 4 * g);
    }
    int rows = 0;
    constexpr int STEP = SPLIT ? 4 : 1;          // as above
    const int start = SPLIT ? wave : 0;
    constexpr int LOADS = R::per_wave / 8;
    RowWalk<LOADS> walk;                         // rows that this lane brings
    RowWalk<1> stat_walk;                        // row whose statistics it brings
    int last = 0;                                // of the list
    auto rewind = [&]() {
        walk.start(KB * start + (SHARED ? 16 * wave : 0) + lane / 8, 8, KB * STEP, n, n_inv);
        stat_walk.start(KB * start + lane % KB, 0, KB * STEP, n, n_inv);
    };
    const unsigned piece = 16 * ((lane % 8) ^ (lane / 8)), my_lds = lds_address(mine) + (SHARED ? 2048 * wave : 0), my_stat_lds = lds_address(my_stats);
    auto request = [&](int local) {
        const int blk = STEP * local + start;
        const unsigned to = my_lds + (local % 2) * (2 * R::buf), st = my_stat_lds + (local % 2) * (4 * kStats);
        auto token = [&](int row) {
            const int r = min(KB * blk + row, rows - 1), p = divide(r, n, n_inv);
            return list[p] + at.slot(r - p * n);
        };
        const bool tables = MODE == kWaves || LCE || walks;
        lds_reads_done();
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            if (tables) {
                const unsigned off = row_offset(walk.token(u, list, last, slots), C, piece);
                load_to_lds_untracked(A.Q + img, off, to + 1024 * u);
                load_to_lds_untracked(A.dO + img, off, to + KB * 128 + 1024 * u);
            } else {
                const size_t e = img + (size_t)token((SHARED ? 16 * wave : 0) + 8 * u + lane / 8) * C + piece / 2;
                load_to_lds_untracked(A.Q + e, to + 1024 * u);
                load_to_lds_untracked(A.dO + e, to + KB * 128 + 1024 * u);
            }
        }
        // statistics: 64 floats per load, (head, lse or D) by wavefront or (lse | D) of one head
        const int t = tables ? stat_walk.token(0, list, last, slots) : token(lane % KB);
        if (SHARED) {
            if (wave < 2 * HPW)
                load4_to_lds_untracked((wave % 2 ? A.dsum : A.lse) + stat0 + (size_t)(wave / 2) * D.N + t, st + 4 * wave * KB);
        } else {
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh)
                load4_to_lds_untracked((lane >= KB ? A.dsum : A.lse) + stat0 + (size_t)hh * D.N + t, st + 8 * hh * KB);
        }
        walk.advance();
        stat_walk.advance();
    };
    auto block = [&](int local) {
        const int blk = STEP * local + start;
        const bf16_t *Qs = mine + (local % 2) * R::buf, *Gs = Qs + KB * 64;
        const float *st = my_stats + (local % 2) * kStats;
#pragma unroll(LCE ? 1 : KB / 32)
        for (int tp = 0; tp < KB / 32; ++tp) {
            const int left = rows - KB * blk - 32 * tp;
            if (tp && left <= 0) break;
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                f32x4 s[NK][2], dp[NK][2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int row = 32 * tp + 16 * t;
                    const f32x4 l4 = *(const f32x4 *)(st + 2 * hh * KB + row + 4 * g);
                    const f32x4 d4 = *(const f32x4 *)(st + (2 * hh + 1) * KB + row + 4 * g);
                    bf16x8 qf[KSD], gf[KSD];
#pragma unroll
                    for (int ks = 0; ks < KSD; ++ks) {
                        qf[ks] = row_operand(Qs, row + i, HD / 8 * hh + 4 * ks + g);
                        gf[ks] = row_operand(Gs, row + i, HD / 8 * hh + 4 * ks + g);
                    }
#pragma unroll
                    for (int q = 0; q < NK; ++q) {
                        s[q][t] = -l4;
                        dp[q][t] = -d4;
#pragma unroll
                        for (int ks = 0; ks < KSD; ++ks) {
                            s[q][t] = mfma16(qf[ks], kf[q][hh][ks], s[q][t]);       // S[query 16 t + 4 g + j][key i]
                            dp[q][t] = mfma16(gf[ks], vf[q][hh][ks], dp[q][t]);
                        }
                    }
                }
                bf16x8 pb[NK], db[NK];
#pragma unroll
                for (int q = 0; q < NK; ++q) {
                    if (left < 32) {
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                if (16 * t + 4 * g + j >= left) s[q][t][j] = -INFINITY;
                    }
                    float p[8], ds[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        p[e] = __builtin_amdgcn_exp2f(s[q][e / 4][e % 4]);
                        ds[e] = p[e] * dp[q][e / 4][e % 4];
                    }
                    pb[q] = pack8(p);
                    db[q] = pack8(ds);
                }
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const bf16x8 gc = column_operand(Gs, 32 * tp, HD * hh + 16 * dt, g, i);
                    const bf16x8 qc = column_operand(Qs, 32 * tp, HD * hh + 16 * dt, g, i);
#pragma unroll
                    for (int q = 0; q < NK; ++q) {
                        dv[q][hh][dt] = mfma16(gc, pb[q], dv[q][hh][dt]);
                        dk[q][hh][dt] = mfma16(qc, db[q], dk[q][hh][dt]);
                    }
                }
                if (SHARED) __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    const int entries = D.R * D.k;
    const int32_t *irb = A.Ir + (size_t)b * entries;
    for (int e0 = 0; e0 < entries;) {
        int named;
        if (SHARED) {
            __syncthreads();                      // the list and the buffers have been read
            named = list_of_group(irb, entries, e0, reg, D.R, k_inv, at, list, counts);
            e0 += kListShared;
            __syncthreads();
        } else {
            named = list_of_wave(irb, entries, e0, reg, D.R, k_inv, at, list);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        }
        rows = named * n;
        last = named - 1;
        rewind();
        const int nb = ((rows + KB - 1) / KB - start + STEP - 1) / STEP;
        if (nb <= 0) continue;
        // the operands have arrived: see above
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) asm volatile("" : "+v"(kf[q][hh][ks]), "+v"(vf[q][hh][ks]));
        request(0);
#pragma unroll 1
        for (int s = 0; s < nb; ++s) {
            const bool more = s + 1 < nb;
            if (SHARED) {
                arrive_barrier();
                if (more) request(s + 1);
            } else if (more) {
                request(s + 1);
                if (HPW == 2) asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if (!idle) block(s);
        }
    }
    // With the pass, LCE^T(dO) is there in float32: its upper halves where dV goes, its lower ones where dK goes.
    auto store = [&](bf16_t *at, f32x4 k, f32x4 v) {
        if (!LCE && lce_blocks) {
            const u32x2 hi = *(const u32x2 *)(at + C), lo = *(const u32x2 *)at;
            v += __builtin_bit_cast(f32x4, u32x4{pair_lo(lo[0], hi[0]), pair_hi(lo[0], hi[0]), pair_lo(lo[1], hi[1]), pair_hi(lo[1], hi[1])});
        }
        *(u32x2 *)at = pack4(k * kLn2);
        *(u32x2 *)(at + C) = pack4(v);
    };
    if constexpr (SPLIT) {
        // wavefront w adds up and stores channels 16 w .. 16 w + 15 of both
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                float *part = sums + ((q * 4 + a) * 8 + wave) * 256 + 4 * lane;
                *(f32x4 *)part = dk[q][a / NDT][a % NDT];
                *(f32x4 *)(part + 1024) = dv[q][a / NDT][a % NDT];
            }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NK; ++q) {
            if (q0 + 16 * q + i >= n) continue;
            const float *part = sums + (q * 4 + wave) * 2048 + 4 * lane;
            bf16_t *dst = A.dQKV + ((size_t)b * D.N + tok[q]) * 3 * C + C + 64 * cg + 16 * wave + 4 * g;
            f32x4 sum[2];
#pragma unroll
            for (int u = 0; u < 2; ++u, part += 1024)
                sum[u] = (*(const f32x4 *)part + *(const f32x4 *)(part + 256)) + (*(const f32x4 *)(part + 512) + *(const f32x4 *)(part + 768));
            store(dst, sum[0], sum[1]);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < NK; ++q) {
        if (q0 + 16 * q + i >= n) continue;
        bf16_t *row = A.dQKV + ((size_t)b * D.N + tok[q]) * 3 * C + C + 64 * cg + 4 * g;
#pragma unroll
        for (int hh = 0; hh < HPW; ++hh)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) store(row + HD * hh + 16 * dt, dk[q][hh][dt], dv[q][hh][dt]);
    }
}

template <int HD, int N, Mode MODE, bool LCE = false>
int launch_t(const Dims &D, const AttnBwdArgs &A, const lce::BackwardJobs &L, int kernel_id, hipStream_t st)
{
    const int per_tile = (MODE == kShared ? 64 : 16) * N, tiles = (D.n + per_tile - 1) / per_tile;
    const long items = (long)D.B * D.R * tiles * (D.C / 64), blocks = ((MODE == kWaves ? (items + 3) / 4 : items) + 7) / 8 * 8;
    if (blocks > 0x7fffffffL / 4) return BRA_ERR_UNSUPPORTED;
    // The pass with the tap gradients is in front where the attention takes several rounds of workgroups, behind where all of it
    // is resident at once (2 x 128 x 128 x 64, k = 4, 512 workgroups: query side 48.5 us with the pass behind, 63 in front;
    // 64 x 56 x 56 x 64, k = 1, 3136 workgroups: 64.5 behind, 55.4 in front, 70 with the two kinds in turn).  The other pass is
    // always behind: its many short workgroups fill up the last round (12 x 112 x 120 x 64, k = 1: key side 76 us, in front 87).
    const bool front = blocks > 768;
    const long with_q = L.beside || LCE ? L.grad.blocks() : 0, with_kv = L.beside && !LCE ? L.add.blocks() : 0;
    const int halo = LCE ? lce::RegionHalo(D.rh, D.rw).bytes(D.n) : 0;
    // kWaves has at most 32 tokens per region and always walks (up to 4096 regions)
    const size_t tables = MODE == kShared ? 1 : 4;
    const int walks = MODE == kSplit ? walk_ok(D) && D.n <= 256 : walk_ok(D);
    auto query_side = [&](auto single) {
        ProfScope ps(st, kernel_id);
        hipLaunchKernelGGL((k_attn_bwd_q<HD, N, MODE, LCE, decltype(single)::value>), dim3((unsigned)(blocks + with_q)), dim3(256),
                           halo + tables * (D.k + (walks ? D.n : 0)) * sizeof(int), st, A, D, tiles, (int)items, walks, L.grad, (int)with_q, front);
    };
    if constexpr (LCE) {
        query_side(std::true_type{});
    } else if constexpr (MODE == kWaves) {
        if (D.kn <= Rows<MODE>::KB) query_side(std::true_type{});
        else query_side(std::false_type{});
    } else {
        query_side(std::false_type{});
    }
    if (hipGetLastError() != hipSuccess) return BRA_ERR_LAUNCH;
    ProfScope ps(st, kernel_id);
    hipLaunchKernelGGL((k_attn_bwd_kv<HD, N, MODE, LCE>), dim3((unsigned)(blocks + with_kv)), dim3(256), tables * (walks ? D.n : 0) * sizeof(int), st, A, D, tiles,
                       (int)items, walks, L.add, (int)with_kv);
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

long wave_groups(const Dims &D) { return (long)D.B * D.R * (D.C / 64); }

// Two token tiles per wavefront (every operand read serves both) where they leave no more than an eighth of their
// tokens empty beyond the narrow ones and there are workgroups enough.
bool two_tiles(const Dims &D)
{
    const long t64 = (D.n + 63) / 64, t128 = (D.n + 127) / 128;
    return t128 * 128 * 8 <= t64 * 64 * 9 && wave_groups(D) * t128 >= 512;
}

// A workgroup has its region whole and all routed keys in one block, and the key side's buffers hold the halo.
// Regions that items of 4 x 4 fill badly only where there are many: whole gradient (us), passes / so, by regions: 6 x 6 tokens (42 x 42 x 64) 392 46.1 / 48.6, 784
// 57.6 / 60.3, 1568 86.3 / 83.4; 3 x 16 784 62.0 / 65.1, 1568 95.5 / 91.3; 4 x 10 320 43.0 / 44.7, 2048 105.4 / 101.2; 8 x 8 392 57.4 / 56.8, 784 76.1 / 74.4.
bool convolves(const Dims &D, const lce::BackwardJobs &L)
{
    const lce::RegionHalo halo(D.rh, D.rw);
    return L.fit && D.n <= 64 && (D.n > 56 || (long)D.B * D.R > 1024) && D.kn <= Rows<kShared>::KB && walk_ok(D) && halo.items() <= 4 * kLceRounds &&
           halo.bytes(D.n) <= 2 * Rows<kShared>::buf * (int)sizeof(bf16_t);
}

Mode mode_of(const Dims &D)
{
    const long waves = wave_groups(D) * (D.n <= 32 ? 1 : 4 * ((D.n + 63) / 64));
    // Too few wavefronts for the 1024 SIMDs: four share the rows of a tile, where a row list has at least two blocks
    // (us for the whole gradient: 3 x 14 x 49 x 64, k = 20: 66 -> 50; 28 x 28 x 64, k = 4, 64 routed keys: 45 -> 42; but
    // 392 wavefronts and 80 keys: 66 -> 69, 196 and 4 keys: 49 -> 60).
    if (waves <= 256 && D.kn >= 64) return kSplit;
    return D.n <= 32 ? kWaves : kShared;
}

template <int HD>
int launch_hd(const Dims &D, const AttnBwdArgs &A, const lce::BackwardJobs &L, int kernel_id, hipStream_t st)
{
    switch (mode_of(D)) {
    case kSplit: return D.n <= 16 ? launch_t<HD, 1, kSplit>(D, A, L, kernel_id, st) : launch_t<HD, 2, kSplit>(D, A, L, kernel_id, st);
    case kWaves: return D.n <= 16 ? launch_t<HD, 1, kWaves>(D, A, L, kernel_id, st) : launch_t<HD, 2, kWaves>(D, A, L, kernel_id, st);
    default:
        if (two_tiles(D)) return launch_t<HD, 2, kShared>(D, A, L, kernel_id, st);
        return convolves(D, L) ? launch_t<HD, 1, kShared, true>(D, A, L, kernel_id, st) : launch_t<HD, 1, kShared>(D, A, L, kernel_id, st);
    }
}

}  // namespace

bool attn_bwd_convolves(const Dims &D, const lce::BackwardJobs &L) { return mode_of(D) == kShared && !two_tiles(D) && convolves(D, L); }

int launch_attn_bwd(const Dims &D, const AttnBwdArgs &A, const lce::BackwardJobs &L, int kernel_id, hipStream_t st)
{
    return D.d == 32 ? launch_hd<32>(D, A, L, kernel_id, st) : launch_hd<64>(D, A, L, kernel_id, st);
}

}  // namespace bra
