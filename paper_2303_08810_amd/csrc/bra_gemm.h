// bf16 products of the general pipelines (bra_gemm.hip; internal).
#pragma once

#include "bra_mfma_dev.h"

namespace bra {

// Rows are the tokens of Hp x Wp maps of which only the top-left H x W part exists in memory (Hp = 0: they all do).
struct GemmRows {
    int Hp = 0, Wp = 0, H = 0, W = 0;
};

// Where a product goes: output column o to buffer o / cols (up to three buffers of `cols` columns each, e.g. Q, K, V),
// column o % cols; cols is a multiple of 8.
struct GemmOut {
    void *buf[3];
    int cols;
    float *f32[2];      // optional float32 copies of the results that go to buf[0] and buf[1] (bf16 output only)
    // bf16 output only, all optional: bias[o] is added, then GELU is applied, then res[m][o]
    // (the layout of buf[0]) is added.
    const float *bias;
    const bf16_t *res;
    int gelu;
    float scale0 = 1.0f;        // bf16 output only: factor of what goes to buf[0] (not of its float32 copy)
    GemmRows in_rows, out_rows; // bf16 output only: missing rows of In read as zeros, missing rows of the buffers are not written
};

// A second product with the same W and K whose input is float32 and enters as three exact bf16 terms, with float32
// results: the region-level projection Q^r | K^r = Xr [Wq | Wk] in the launch of the token projection.
struct GemmRegions {
    const float *In;
    long M;
    int Nout;
    float *buf[2];
    int cols;
};

// Rows of In and of the output taken region by region (n tokens each, row-major within the region) of maps of S x S regions of
// rh x rw tokens, of which In holds the top-left H x W part (the rest reads as zeros), and float32 means over each region's tokens of the results that
// go to buf[0] and buf[1] of the output, before they are rounded and scaled.  An output buffer that is NULL is not written.
struct GemmMeans {
    float *buf[2];
    int regions, R, S, n, rh, rw, H, W;
    float n_inv, R_inv, S_inv, rw_inv;
};
// Tiles hold whole regions: not of more tokens than the smallest tile has rows.
constexpr int kMeansMaxTokens = 64;

// Out = In W: In [M, K] bf16, W row-major [K][ldw]; K a multiple of 64, Nout of 8.
int gemm(const bf16_t *In, const bf16_t *W, int ldw, long M, int K, int Nout, const GemmOut &out, const GemmRegions *regions,
         int kernel_id, hipStream_t st);
// The same over the regions of a map, with their means; K <= 4096.
int gemm_means(const bf16_t *In, const bf16_t *W, int ldw, int K, int Nout, const GemmOut &out, const GemmMeans &means, int kernel_id, hipStream_t st);
// Out = In Wt^T: Wt [Nout][ldw], the contraction axis contiguous.
int gemm_bt(const bf16_t *In, const bf16_t *Wt, int ldw, long M, int K, int Nout, bf16_t *Out, int kernel_id, hipStream_t st);

// Out = In W and Out = In Wt^T (b.W is Wt) over the same M rows and contraction, in one launch.
struct GemmHalf {
    const bf16_t *In, *W;
    int ldw, Nout;
    GemmOut out;
};
int gemm_pair(const GemmHalf &a, const GemmHalf &b, long M, int K, int kernel_id, hipStream_t st);

// Contractions over all M tokens: Part[share][KA][N] = A^T B over the share's tokens, for two products in one launch with
// gemm_tn_shares(M, ..) shares each (their sum, in a fixed order, is the product).  Sizes and pitches multiples of 8.
struct GemmTn {
    const bf16_t *A, *Bm;
    float *Part;
    int lda, ldb, KA, N;
};
int gemm_tn_shares(long M, int KA0, int N0, int KA1, int N1);
int gemm_tn(const GemmTn &J0, const GemmTn &J1, long M, int kernel_id, hipStream_t st);

// The same and b: Out = In Wt^T over the M rows into one buffer, a contraction of K > 64; small ones in one launch.
int gemm_bt_tn(const GemmTn &J0, const GemmTn &J1, const GemmHalf &b, long M, int K, int kernel_id, hipStream_t st);

// The region-level product on its own.
int gemm_regions(const GemmRegions &r, const bf16_t *W, int ldw, int K, int kernel_id, hipStream_t st);

}  // namespace bra
