// Attention of bf16 models with 64-wide heads (attention_mfma.h).
#include "attention_mfma.h"

namespace kvr {

hipError_t launch_attention_mfma64(const bf16_t *Q, const bf16_t *Q_lo, const RowInfo *rows, const AttnItem *items,
                                   int n_items, int MT, int layer, int Hq, int Hkv, float *part, bf16_t *O, bf16_t *O_lo,
                                   bool o_perm, float *lse, hipStream_t s) {
    return launch_mfma_hd<64>(Q, Q_lo, rows, items, n_items, MT, layer, Hq, Hkv, part, O, O_lo, o_perm, lse, s);
}

}  // namespace kvr
