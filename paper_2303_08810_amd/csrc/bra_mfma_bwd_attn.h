// Attention backward over regions of any size (bra_mfma_bwd_attn.hip; internal).
#pragma once

#include "bra_lce_pairs.h"

namespace bra {

struct AttnBwdArgs {
    const bf16_t *Q, *K, *V, *dO;      // [B N, C]; Q multiplied by scale log2(e)
    const int32_t *Ir;
    bf16_t *O, *dQKV;                  // [B N, C] attention output, [B N, 3C] gradients
    float *lse, *dsum;                 // [B][heads][N] row statistics
};

// With lce.beside, or where attn_bwd_convolves(), both passes of lce are done within the two launches; without, the caller runs them afterwards.
bool attn_bwd_convolves(const Dims &D, const lce::BackwardJobs &lce);
int launch_attn_bwd(const Dims &D, const AttnBwdArgs &A, const lce::BackwardJobs &lce, int kernel_id, hipStream_t st);

}  // namespace bra
