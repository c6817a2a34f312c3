// Internal: the attention kernel of ff_attn_rows.hip as ff_mfma.hip launches it.
#pragma once

#include "ff_common.h"

#include <type_traits>

namespace ff {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// Sum of the lane's own four bf16 values (w0, w1), added to every element of acc: a 4 x 4 x 4 matrix instruction (sixteen
// independent blocks of four lanes) against ones.
__device__ __forceinline__ f32x4 add_four(uint32_t w0, uint32_t w1, f32x4 acc) {
    const i16x4 ones = __builtin_bit_cast(i16x4, make_uint2(0x3f803f80u, 0x3f803f80u));
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(i16x4, make_uint2(w0, w1)), acc, 0, 0, 0);
}
// -inf for the keys of a tile of S^T whose bit in live is not set: one more contraction step, the key side 0 or -inf against a
// one.  kperm: key of the lane's row of S^T, hf: half-wave
__device__ __forceinline__ f32x16 mask_step(uint32_t live, int kperm, int hf, f32x16 s) {
    const uint32_t term = (live >> kperm) & 1u ? 0u : 0x0000ff80u;
    const i16x4 k_mask = __builtin_bit_cast(i16x4, make_uint2(hf == 0 ? term : 0u, 0u));
    const i16x4 q_one = __builtin_bit_cast(i16x4, make_uint2(hf == 0 ? 0x00003f80u : 0u, 0u));
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(k_mask, q_one, s, 0, 0, 0);
}

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
