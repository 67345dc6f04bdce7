// Image-resident attention backward (bra_mfma_bwd_map.hip; internal).
#pragma once

#include "bra_common.h"

namespace bra {

bool attn_bwd_map_ok(const Dims &D);
// The depth-wise parts are in the launch: O and dV with LCE(V) and LCE^T(dO), and the tap gradients of each image as PartLce [B][C][25].
bool attn_bwd_map_convolves(const Dims &D);
// Attention output into O [B N, C], dQ | dK | dV into dQKV [B N, 3C].
int launch_attn_bwd_map(const Dims &D, const bf16_t *Q, const bf16_t *K, const bf16_t *V, const bf16_t *dO, const int32_t *Ir,
                        bf16_t *O, bf16_t *dQKV, const bf16_t *Wlce, float *PartLce, int kernel_id, hipStream_t st);

}  // namespace bra
