// Internal: the attention kernel of ff_attn_rows.hip as ff_mfma.hip launches it.
#pragma once

#include "ff_common.h"

#include <type_traits>

namespace ff {

struct AttnRowsArgs {
    const bf16_t *q, *k, *g, *vt;   // q, k, gate [rows][H][Lp][d]; v^T [rows][H][Lp/32][d][32]
    bf16_t* o;                      // gated context [rows][H][Lp][d]
    const float* bias;              // 32 x 32 tiles in accumulator order (bias_index of ff_mfma.hip), or NULL
    const float* mask;              // caller's mask or NULL
    int64_t sr, sl;                 // mask strides
    int r0, rows, L, Lp, Lq, H;
    int n_items, n_rb, n_qb;        // filled in by the launch: work items, row blocks, query blocks
};
ff_status attn_rows_launch(const AttnRowsArgs& a, int d, hipStream_t st);      // d: head dimension, 8, 16 or 32

}  // namespace ff
