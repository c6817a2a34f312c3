// Internal: the attention kernel of ff_attn_rows.hip as ff_mfma.hip launches it, and the device code that it shares with
// k_proj_attn there.
#pragma once

#include "ff_common.h"

#include <type_traits>

namespace ff {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

union Frag {
    bf16x8 v;
    uint4 u;
    uint32_t w[4];
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {   // a -> low half (first element)
    bf16x2 t;
    t[0] = (__bf16)a;
    t[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, t);
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// A load with the address split into a wave-uniform base (scalar registers) and a 32-bit byte offset per lane: one
// instruction, no address arithmetic in the vector unit.
__device__ __forceinline__ uint4 ldg16(const void* base, uint32_t lane_bytes) {
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(base) + lane_bytes);
}

// sum of the two bf16 halves of w, added to acc (v_dot2c_f32_bf16)
__device__ __forceinline__ float add_pair(uint32_t w, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, 0x3f803f80u), acc,
                                           false);
}

// value of the other half-wave's lane (l ^ 32)
__device__ __forceinline__ float other_half(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    // r[0] = {lower half of v, lower half of v}, r[1] = {upper half, upper half}
    return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

// After the call lanes of the lower half hold (a of lower lane, a of upper lane) and lanes of
// the upper half hold (b of lower lane, b of upper lane): two 4-element groups that are
// adjacent in memory end up in one lane.
__device__ __forceinline__ void merge_halves(uint32_t& a, uint32_t& b) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

constexpr int kWaitVmcnt0 = 0x0F70;      // s_waitcnt vmcnt(0), the other counters untouched

// Sums over a piece of P^T as the 32 x 32 x 16 instructions hold it (lane = query, the lower half-wave the keys 0 .. 7, the upper 8 .. 15), added to acc: element 0 of
// the result is the sum over both halves for the lane's query.  One 16 x 16 x 32 matrix instruction: it reads the same registers as sixteen columns
// of 32 rows, in which query q % 16 has its keys in the rows 0 .. 7 and 16 .. 23, query 16 + q % 16 in the others; the rows of `sel` select one or the other, so that
// each group of four result rows belongs to the sixteen lanes that hold it.
__device__ __forceinline__ bf16x8 sum_select(int lane) {
    const uint32_t w = (((lane & 15) >> 2) ^ (lane >> 4)) & 1 ? 0u : 0x3f803f80u;
    Frag f;
    f.u = make_uint4(w, w, w, w);
    return f.v;
}
__device__ __forceinline__ f32x4 add_piece(bf16x8 sel, bf16x8 piece, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, piece, acc, 0, 0, 0);
}
// -inf for the keys of a tile of S^T whose bit in live is not set: one more contraction step, the key side 0 or -inf against a
// one.  kperm: key of the lane's row of S^T, hf: half-wave
__device__ __forceinline__ f32x16 mask_step(uint32_t live, int kperm, int hf, f32x16 s) {
    const uint32_t term = (live >> kperm) & 1u ? 0u : 0x0000ff80u;
    const i16x4 k_mask = __builtin_bit_cast(i16x4, make_uint2(hf == 0 ? term : 0u, 0u));
    const i16x4 q_one = __builtin_bit_cast(i16x4, make_uint2(hf == 0 ? 0x00003f80u : 0u, 0u));
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(k_mask, q_one, s, 0, 0, 0);
}

// ---- the softmax of k_attn_rows and k_proj_attn runs without a reference: which results stand, and the general form
// Registers 0 .. N-1 of o hold neither an infinity nor NaN.
template <int N>
__device__ __forceinline__ bool all_finite(const f32x16& o) {
    float z = 0.f;
#pragma unroll
    for (int v = 0; v < N; ++v) z = fmaf(o[v], 0.f, z);
    return z == 0.f;
}
// The lane's query and batch row stand if the denominator lies in [2^-60, 2^96] (else some weights overflowed, or all of them are tiny,
// or one is NaN; 0 is right where no key is attended to, and costs nothing below) and the context is finite (else a value
// overflowed its sum, or a masked key holds NaN or an infinity, which weight 0 does not remove).  N: registers of the context.
template <int N>
__device__ __forceinline__ bool softmax_stands(const f32x16& o, float l_tot) {
    return l_tot >= 0x1p-60f && l_tot <= 0x1p96f && all_finite<N>(o);
}
// Otherwise the row is done again, tile by tile with a running maximum m: scores s of 32 keys, bias included (lane = query, register v = key
// 16 (v / 8) + 8 hf + v % 8), v^T pieces vf (the keys 16 c + 8 hf .. + 7), live: bit = key is attended to.  Nothing that a masked
// key holds reaches a sum; tiles without a live key are left out by the caller.
__device__ __forceinline__ void general_tile(f32x16 s, Frag (&vf)[2], uint32_t live, int hf, f32x16& o, float& m, float& l) {
    if (live != 0xffffffffu) {
        const uint32_t mine = live >> (8 * hf);
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = (mine >> (16 * (v >> 3) + (v & 7))) & 1u ? s[v] : -INFINITY;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t two = mine >> (16 * c + 2 * i);
                vf[c].w[i] &= ((two & 1u) ? 0xffffu : 0u) | ((two & 2u) ? 0xffff0000u : 0u);
            }
    }
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    const float m_new = fmaxf(m, fmaxf(mx, other_half(mx)));
    const float ref = m_new == -INFINITY ? 0.f : m_new, sc = __builtin_amdgcn_exp2f(m - ref);
    m = m_new;
    l *= sc;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] *= sc;
    Frag p[2];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        p[g >> 2].w[g & 3] = pack2(__builtin_amdgcn_exp2f(s[2 * g] - ref), __builtin_amdgcn_exp2f(s[2 * g + 1] - ref));
        l = add_pair(p[g >> 2].w[g & 3], l);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c].v, p[c].v, o, 0, 0, 0);
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
