// Generic kernel family: every step of the gated attention with float32 accuracy, for any shape and for both storage types.  It
// is the float32 path (nothing is held in fewer bits when T = float) and the fallback for bfloat16 shapes the bfloat16
// matrix-core family does not take.  Steps follow FastFold Section 2.1 (projections, scaled dot product, softmax,
// product with V, output linear), Section 2.3 (axes, pair bias) and Section 5.2 (softmax with the mask and bias
// addends fused in; gate = bias + sigmoid + product).
//
// All contractions run on the bfloat16 matrix instruction v_mfma_f32_32x32x16_bf16, a float32 operand as the exact sum of three bfloat16 values
// (see split4), a bfloat16 one as it is.  Operand layouts (wave64): A (32 x 16): lane l holds row l%32, columns 8*(l/32) .. + 7; B (16 x 32): lane l
// holds column l%32, rows 8*(l/32) .. + 7; C/D (32 x 32): lane l holds column l%32, register v holds row 8*(v/4) + 4*(l/32) + v%4.
// Measured (row attention, 64 x 155 tokens of 256 channels, 8 heads of 32, 8.1 GFLOP): 1.40 ms with vector
// multiply-adds, a wavefront per query and per pair, 0.116 ms on v_mfma_f32_32x32x2_f32 (whose matrix cores alone need 53 us), 0.090 ms so (kernels under the
// profiler: projections 42 to 47 us, attention 25 to 28, output projection 17 to 19, rows 9 to 10); relative error against float64 3.9e-7 -> 2.3e-7, and 0.48 to 0.90 of the
// float32 instruction's in each of 508 other shapes of 4 to 3000 channels and head dims 4 to 128.  Where the planes do not reach, the float32 instruction takes over
// (float32_tile, float32_queries).
//
// Workspace layout of this family, per chunk of `rows` batch rows, token t = rl*L + l:
//   stats [tokens][2]   float32 mean, 1/std of LayerNorm
//   qkvg  [tokens][4*Hd] T : q (times log2(e)/sqrt(d)), k, v, sigmoid gate
//   o     [tokens][Hd]   T : gate * context; until the attention writes it, the planes of the projection weights (weight_planes)
//   bias  [H][L][Lb]     float32, times log2(e); rows padded to a multiple of four (16-byte reads)
#include "ff_attn_rows.h"
#include "ff_common.h"

#include <type_traits>

namespace ff {
namespace gen {

static inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline int bias_pitch(int L) { return (L + 3) & ~3; }

__device__ __forceinline__ float4 keep4(bool on, const float4& v) {      // v or zeros, component by component
    return make_float4(on ? v.x : 0.f, on ? v.y : 0.f, on ? v.z : 0.f, on ? v.w : 0.f);
}

// Elements k .. k + 3 of a row of n elements, zeros beyond n, in two steps: the access, and what is done with its result
// once it is needed (anything done with a loaded value right away is a wait for it).  VEC: n is a multiple of four and
// the row aligned to four elements, so that they are one access, without a condition on it (a branch and a wait of its
// own): a piece beyond the row reads the last one and drops it.
template <typename T, bool VEC>
struct Piece {
    float4 v;
    __device__ __forceinline__ void fetch(const T* row, int k, int n) {
        v.x = k < n ? to_f32<T>(row[k]) : 0.f;
        v.y = k + 1 < n ? to_f32<T>(row[k + 1]) : 0.f;
        v.z = k + 2 < n ? to_f32<T>(row[k + 2]) : 0.f;
        v.w = k + 3 < n ? to_f32<T>(row[k + 3]) : 0.f;
    }
    __device__ __forceinline__ float4 value(int, int) const { return v; }
};
template <>
struct Piece<float, true> {
    float4 v;
    __device__ __forceinline__ void fetch(const float* row, int k, int n) { v = *reinterpret_cast<const float4*>(row + (k < n ? k : n - 4)); }
    __device__ __forceinline__ float4 value(int k, int n) const { return keep4(k < n, v); }
};
template <>
struct Piece<bf16_t, true> {
    uint2 v;
    __device__ __forceinline__ void fetch(const bf16_t* row, int k, int n) { v = *reinterpret_cast<const uint2*>(row + (k < n ? k : n - 4)); }
    __device__ __forceinline__ float4 value(int k, int n) const {
        return keep4(k < n, make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                                        __uint_as_float(v.y & 0xffff0000u)));
    }
};
// (rows of whole pieces only: neither clamped nor cleared)
template <typename T>
struct WholePiece {
    Piece<T, true> p;
    __device__ __forceinline__ void fetch(const T* row, int k, int) { p.v = *reinterpret_cast<const decltype(p.v)*>(row + k); }
    __device__ __forceinline__ float4 value(int, int) const { return p.value(0, 1); }
};
template <typename T, bool VEC>
__device__ __forceinline__ float4 load4(const T* row, int k, int n) {
    Piece<T, VEC> p;
    p.fetch(row, k, n);
    return p.value(k, n);
}
template <typename T, bool VEC>
__device__ __forceinline__ void store4(T* row, int k, int n, const float4& v) {
    if constexpr (VEC) {
        if (k < n) {
            if constexpr (sizeof(T) == 4)
                *reinterpret_cast<float4*>(row + k) = v;
            else
                *reinterpret_cast<uint2*>(row + k) =
                    make_uint2(f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16), f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16));
        }
    } else {
        if (k < n) row[k] = from_f32<T>(v.x);
        if (k + 1 < n) row[k + 1] = from_f32<T>(v.y);
        if (k + 2 < n) row[k + 2] = from_f32<T>(v.z);
        if (k + 3 < n) row[k + 3] = from_f32<T>(v.w);
    }
}

// ---------------------------------------------------------------------------------------
// Float32 contractions on the bfloat16 matrix instruction.  A float32 value is the exact sum of three bfloat16 values (8 + 8 + 8 significant bits,
// each the rounding of what the ones before it left): x = x0 + x1 + x2, |x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|.  Of the nine products of two such
// sums the six with i + j <= 2 are formed; what is left out is at most 2^-24 (1 + 2^-10) of the product, as much as one float32 rounding of it (x = y = 0x1.00ff8p0: 2^-24.0),
// and 2^-27.4 in the root mean square of normal values, of either sign.  x0 y0 and the five corrections have sums of their own, so a chain rounds once per 16 terms of the contraction (v_mfma_f32_32x32x2_f32: once per two).
// Six instructions of 32 cycles for 16 terms against eight of 64.  A bfloat16 operand is one plane and needs no others.
// The operands are taken times 2^24, exactly, so that the third plane of the smallest float32 lies inside the range of bfloat16 too (unscaled, operands below
// 2^-109 lose their last bits: relative error 3e-4 at 2^-120 instead of 2e-7).  An infinite one, or one that overflows so (from 2^104 on), has NaN in its lower planes: results that are not finite are formed again by the float32
// instruction (float32_tile, float32_queries).
constexpr float kUp = 0x1p24f, kDown = 0x1p-24f;
__device__ __forceinline__ float4 times4(const float4& v, float f) { return make_float4(v.x * f, v.y * f, v.z * f, v.w * f); }
// The same of a piece whose loads are under conditions (VEC false): opaque, or the compiler moves the product to the load, where it waits for it (rows of no
// whole pieces took 16 % longer)
template <bool VEC>
__device__ __forceinline__ float4 times4_piece(float4 v, float f) {
    if constexpr (!VEC) asm("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
    return times4(v, f);
}
template <int NP>
struct Planes {
    uint2 p[NP];       // four elements in each
};
template <int NP>
__device__ __forceinline__ Planes<NP> split4(const float4& v) {
    Planes<NP> s;
    float4 r = v;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        s.p[i] = make_uint2(pack2(r.x, r.y), pack2(r.z, r.w));
        asm("" : "+v"(s.p[i].x));
        asm("" : "+v"(s.p[i].y));      // (else the low halves are rounded once more by themselves)
        if (i + 1 < NP)
            r = make_float4(r.x - lo_f32(s.p[i].x), r.y - hi_f32(s.p[i].x), r.z - lo_f32(s.p[i].y), r.w - hi_f32(s.p[i].y));
    }
    return s;
}
// hi += x0 y0 and lo += the corrections, 16 terms of the contraction (lo of a single product stays as it is)
template <int NA, int NB>
__device__ __forceinline__ void mfma_split(const Frag (&x)[NA], const Frag (&y)[NB], f32x16& hi, f32x16& lo) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (i + j > 0 && i + j <= 2) lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i].v, y[j].v, lo, 0, 0, 0);
    hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0].v, y[0].v, hi, 0, 0, 0);
}

// ---------------------------------------------------------------------------------------
// LayerNorm rows: pair bias and token statistics in one launch.  Eight lanes per row, lane j of them with the
// elements 4j + 32i .. + 3: a row of 32 elements is one line, and a sum over a row three exchanges instead of the six
// of a wavefront per row (which spent most of its time on them: H + 2 sums per pair).  Rows of up to 256 elements
// stay in registers (NJ pieces per lane); NJ = 0 reads longer ones again for every pass.
//   pairs [0, L*L):  bias[h][q][k] = log2(e) * sum_c LN(src[(q*sq + k*sk)*c ...])_c * w_b[h][c]
//   then the tokens of the chunk: mean and 1/std into stats
struct RowsArgs {
    const void* src;           // pairs
    int64_t sq, sk;
    int cp;                    // channels of a pair
    const void *g, *b, *wb;    // LayerNorm of the pairs, bias weights [H][cp]
    int H, L, Lb;
    float* bias;
    int pair_blocks;           // blocks (32 rows each) of the pairs; 0: no bias
    const void* x;             // tokens: (r, l) at x + ((r0 + r)*sr + l*sl)*c
    int64_t sr, sl;
    int c, r0, tokens;
    float* stats;
    float eps;
    const void* w[4];          // w_q, w_k, w_v, w_g [Hd][c], to be split into planes (see weight_planes)
    int Hd, token_blocks;
    unsigned char* planes;
};

template <typename T, bool VEC, int NJ>
__device__ __forceinline__ void row_stats(const T* row, int c, int j8, float eps, float& mean, float& rstd, float4 (&reg)[NJ > 0 ? NJ : 1]) {
    float s = 0.f, q = 0.f;
    auto passes = [&](auto&& f) {
        if constexpr (NJ > 0) {
#pragma unroll
            for (int i = 0; i < NJ; ++i) f(reg[i], 4 * j8 + 32 * i);
        } else {
            for (int k = 4 * j8; k < c; k += 32) f(load4<T, VEC>(row, k, c), k);
        }
    };
    if constexpr (NJ > 0) {
#pragma unroll
        for (int i = 0; i < NJ; ++i) reg[i] = load4<T, VEC>(row, 4 * j8 + 32 * i, c);
    }
    passes([&](const float4& v, int) { s += (v.x + v.y) + (v.z + v.w); });
    mean = sum8(s) / (float)c;
    passes([&](const float4& v, int k) {
        const float a = v.x - mean, b = v.y - mean, d = v.z - mean, e = v.w - mean;
        if (k < c) q += a * a;
        if (k + 1 < c) q += b * b;
        if (k + 2 < c) q += d * d;
        if (k + 3 < c) q += e * e;
    });
    rstd = rsqrtf(sum8(q) / (float)c + eps);
}

template <typename T, bool VEC, int NJ>
__device__ __forceinline__ void pair_row(const RowsArgs& a, int64_t pair, int j8) {
    const bool in = pair < (int64_t)a.L * a.L;
    const int q = in ? (int)(pair / a.L) : 0, k = in ? (int)(pair - (int64_t)q * a.L) : 0;
    const T* row = (const T*)a.src + ((int64_t)q * a.sq + (int64_t)k * a.sk) * a.cp;
    float4 reg[NJ > 0 ? NJ : 1];
    float mean, rstd;
    row_stats<T, VEC, NJ>(row, a.cp, j8, a.eps, mean, rstd, reg);
    auto normal = [&](const float4& v, int i) {
        const float4 g = load4<T, VEC>((const T*)a.g, i, a.cp), b = load4<T, VEC>((const T*)a.b, i, a.cp);
        return make_float4((v.x - mean) * rstd * g.x + b.x, (v.y - mean) * rstd * g.y + b.y, (v.z - mean) * rstd * g.z + b.z,
                           (v.w - mean) * rstd * g.w + b.w);
    };
    if constexpr (NJ > 0) {
#pragma unroll
        for (int i = 0; i < NJ; ++i) reg[i] = normal(reg[i], 4 * j8 + 32 * i);
    }
    for (int h = 0; h < a.H; ++h) {
        const T* w = (const T*)a.wb + (size_t)h * a.cp;
        float acc = 0.f;
        auto add = [&](const float4& x, int i) {
            const float4 wv = load4<T, VEC>(w, i, a.cp);                 // (zeros beyond the row)
            acc += x.x * wv.x;
            acc += x.y * wv.y;
            acc += x.z * wv.z;
            acc += x.w * wv.w;
        };
        if constexpr (NJ > 0) {
#pragma unroll
            for (int i = 0; i < NJ; ++i) add(reg[i], 4 * j8 + 32 * i);
        } else {
            for (int i = 4 * j8; i < a.cp; i += 32) add(normal(load4<T, VEC>(row, i, a.cp), i), i);
        }
        acc = sum8(acc);
        if (in && j8 == (h & 7)) a.bias[((size_t)h * a.L + q) * a.Lb + k] = acc * kLog2e;
    }
}

template <typename T, bool VEC, int NJ>
__device__ __forceinline__ void token_row(const RowsArgs& a, int t, int j8) {
    const bool in = t < a.tokens;
    const int rl = in ? t / a.L : 0, l = in ? t - rl * a.L : 0;
    float4 reg[NJ > 0 ? NJ : 1];
    float mean, rstd;
    row_stats<T, VEC, NJ>((const T*)a.x + ((int64_t)(a.r0 + rl) * a.sr + (int64_t)l * a.sl) * a.c, a.c, j8, a.eps, mean, rstd, reg);
    if (in && j8 == 0) *reinterpret_cast<float2*>(a.stats + 2 * (size_t)t) = make_float2(mean, rstd);
}

// The merged projection weights in the planes of their bfloat16 sums, laid out as the GEMM's LDS image wants them: [chunk of 32 elements][plane][row,
// N rounded up to 128][64 bytes, 16-byte pieces placed as in the GEMM].  Rows beyond N repeat the first one.
__host__ __device__ inline int plane_rows(int n) { return (n + 127) & ~127; }
__device__ __forceinline__ int piece_place(int row, int pc) { return ((((pc >> 1) ^ (row >> 2)) & 3) << 4) + ((pc & 1) << 3); }
__device__ __forceinline__ void split_weights(const RowsArgs& a, int id) {
    const int np = plane_rows(4 * a.Hd), per = a.c >> 2;
    const int row = id / per, p = id - row * per;
    if (row >= np) return;
    const int n = row < 4 * a.Hd ? row : 0, seg = n / a.Hd;
    const float* w = (const float*)(seg == 0 ? a.w[0] : (seg == 1 ? a.w[1] : (seg == 2 ? a.w[2] : a.w[3])));
    const Planes<3> sp = split4<3>(times4(load4<float, true>(w + (size_t)(n - seg * a.Hd) * a.c, 4 * p, a.c), kUp));
#pragma unroll
    for (int j = 0; j < 3; ++j)
        *reinterpret_cast<uint2*>(a.planes + ((size_t)((p >> 3) * 3 + j) * np + row) * 64 + piece_place(row, p & 7)) = sp.p[j];
}

template <typename T, bool VEC>
__device__ __forceinline__ void pair_rows(const RowsArgs& a, int block) {
    const int j8 = threadIdx.x & 7;
    const int64_t pair = (int64_t)block * 32 + (threadIdx.x >> 3);
    if (a.cp <= 32) pair_row<T, VEC, 1>(a, pair, j8);
    else if (a.cp <= 64) pair_row<T, VEC, 2>(a, pair, j8);
    else if (a.cp <= 128) pair_row<T, VEC, 4>(a, pair, j8);
    else if (a.cp <= 256) pair_row<T, VEC, 8>(a, pair, j8);
    else pair_row<T, VEC, 0>(a, pair, j8);
}

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_rows_generic(RowsArgs a) {
    const int j8 = threadIdx.x & 7, r32 = threadIdx.x >> 3;
    if ((int)blockIdx.x < a.pair_blocks) {
        pair_rows<T, VEC>(a, blockIdx.x);
        return;
    }
    if constexpr (sizeof(T) == 4) {
        if ((int)blockIdx.x >= a.pair_blocks + a.token_blocks) {
            split_weights(a, ((int)blockIdx.x - a.pair_blocks - a.token_blocks) * 256 + threadIdx.x);
            return;
        }
    }
    const int t = ((int)blockIdx.x - a.pair_blocks) * 32 + r32;
    if (a.c <= 32) token_row<T, VEC, 1>(a, t, j8);
    else if (a.c <= 64) token_row<T, VEC, 2>(a, t, j8);
    else if (a.c <= 128) token_row<T, VEC, 4>(a, t, j8);
    else if (a.c <= 256) token_row<T, VEC, 8>(a, t, j8);
    else token_row<T, VEC, 0>(a, t, j8);
}

// ---------------------------------------------------------------------------------------
// GEMM, 64 tokens x 64 WN features per block of four wavefronts, contraction in chunks of 32 through double-buffered LDS, the operands split into
// their planes on the way there; a wavefront takes 32 tokens x 32 WN features.
//   PROJ = true : A = LayerNorm(x) on the fly (stats, gamma, beta), B rows from w_q|w_k|w_v|w_g,
//                 epilogue: q scaled, gate = sigmoid(acc + b_g); C -> qkvg[t][4Hd]
//   PROJ = false: A = o[t][Hd], B = w_o, epilogue + b_o, C -> out at the token's address.
// What bounds it (64 x 155 tokens of 256 channels, projections, under the profiler, what a part of the kernel adds to the others): the matrix instructions 12.5 us of 43,
// splitting the tokens 10, the weights' planes 6, loads, stores and a block's beginning and end 15: the waves of a SIMD hide little of one behind another.
// With one buffer and four blocks per compute unit the call takes 84 to 87 us instead of 81 to 84, with the split woven between the matrix instructions 92 (one box).
struct GenericGemmArgs {
    const void* a;         // x (PROJ) or o
    int64_t sr, sl;        // token strides of x / out
    int L, r0, tokens;     // chunk geometry
    int K, N;              // contraction length, output features
    const float* stats;
    const void *ln_g, *ln_b;
    const void* w[4];      // PROJ: w_q, w_k, w_v, w_g ([Hd][K] each); else w[0] = w_o [N][K]
    const void* bvec;      // PROJ: b_g [Hd]; else b_o [N]
    const unsigned char* planes;   // the weights already split (split_weights), or NULL
    int Hd;
    float qscale;
    void* cdst;            // qkvg or out
    const void* res;       // !PROJ: residual added to the output (laid out like out, may be out itself) or NULL
    float eps;             // OWN: of the LayerNorm
};

// 1 / x of a normal x below 2^126: a Newton step in multiply-adds on the instruction's result, which is good to a unit in the last place, rounds correctly (but for a
// significand of ones, half a unit and 2^-25 of it off; Markstein 1990, "Computation of elementary functions on the IBM RISC System/6000 processor").  Divisions take
// 0.9 % more of a call, over 240 shapes.
__device__ __forceinline__ float reciprocal(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.f), r, r);
}

// A tile of 32 tokens x 32 features (lane = feature f0 + lane % 32) whose split sums are not all finite: those elements again, their products formed by the
// float32 instruction (a lane reads four consecutive elements k0 + 4 half .. + 3 of its row of either operand and feeds four instructions
// with them), two sums per output as everywhere.  The finite ones stay, so that an element's bits do not depend on its neighbours'.  Rows whose statistics are
// NaN, and those of the context that begin with a NaN, are NaN by right: what masked tokens hold (their own queries' contexts are NaN throughout) is not worked on.
template <typename T, bool PROJ, bool V>
__device__ __forceinline__ void float32_tile(const GenericGemmArgs& g, int tw, int f0, const float2* own_stats, f32x16& acc) {
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;
    const int t = tw + col < g.tokens ? tw + col : g.tokens - 1;
    const T* row;
    if constexpr (PROJ) {
        const int rl = t / g.L, l = t - rl * g.L;
        row = (const T*)g.a + ((int64_t)(g.r0 + rl) * g.sr + (int64_t)l * g.sl) * g.K;
    } else {
        row = (const T*)g.a + (size_t)t * g.K;
    }
    float2 st = make_float2(0.f, 0.f);
    if constexpr (PROJ) st = own_stats ? own_stats[t - tw] : *reinterpret_cast<const float2*>(g.stats + 2 * (size_t)t);
    const float first = PROJ ? st.y : to_f32<T>(row[0]);
    const uint32_t skip = (uint32_t)__ballot(first != first);            // (the two half-waves hold the same tokens)
    uint32_t redo = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int x = 8 * (v >> 2) + 4 * hf + (v & 3);
        if (!(fabsf(acc[v]) < INFINITY) && tw + x < g.tokens && !((skip >> x) & 1)) redo |= 1u << v;
    }
    const int f = f0 + col < g.N ? f0 + col : g.N - 1;
    if (f0 + col >= g.N) redo = 0;
    if (!__ballot(redo != 0)) return;
    const T* wrow;
    if constexpr (PROJ) {
        const int seg = f / g.Hd;
        const void* w = seg == 0 ? g.w[0] : (seg == 1 ? g.w[1] : (seg == 2 ? g.w[2] : g.w[3]));
        wrow = (const T*)w + (size_t)(f - seg * g.Hd) * g.K;
    } else {
        wrow = (const T*)g.w[0] + (size_t)f * g.K;
    }
    f32x16 even, odd;
#pragma unroll
    for (int v = 0; v < 16; ++v) even[v] = odd[v] = 0.f;
#pragma unroll 1
    for (int k0 = 0; k0 < g.K; k0 += 8) {
        const int k = k0 + 4 * hf;
        float4 a = load4<T, V>(row, k, g.K);
        const float4 w = load4<T, V>(wrow, k, g.K);
        if constexpr (PROJ) {
            const float4 gv = load4<T, V>((const T*)g.ln_g, k, g.K), bv = load4<T, V>((const T*)g.ln_b, k, g.K);
            a = make_float4((a.x - st.x) * st.y * gv.x + bv.x, (a.y - st.x) * st.y * gv.y + bv.y, (a.z - st.x) * st.y * gv.z + bv.z,
                            (a.w - st.x) * st.y * gv.w + bv.w);
        }
        even = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, w.x, even, 0, 0, 0);
        odd = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, w.y, odd, 0, 0, 0);
        even = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, w.z, even, 0, 0, 0);
        odd = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, w.w, odd, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
        if ((redo >> v) & 1) acc[v] = even[v] + odd[v];
}

// BP: weights from g.planes.  VEC: 0 rows of any length, 1 of whole pieces (Piece), 2 of whole chunks.  OWN: the block forms the statistics of its tokens itself
template <typename T, bool PROJ, int VEC, int WN, bool BP, bool OWN>
__device__ __forceinline__ void gemm_block(const GenericGemmArgs& g, int bx, int by) {
    constexpr int BM = 64, BN = 64 * WN;
    constexpr int NA = PROJ || sizeof(T) == 4 ? 3 : 1, NB = sizeof(T) == 4 ? 3 : 1;      // planes of the operands
    constexpr float down = (NA == 3 ? kDown : 1.f) * (NB == 3 ? kDown : 1.f);
    using Load = std::conditional_t<VEC == 2, WholePiece<T>, Piece<T, VEC != 0>>;
    // rows of 32 elements in each plane, 16-byte piece p of row r in place p ^ (r / 4 % 4): conflict-free reads with lane = row
    __shared__ __attribute__((aligned(16))) unsigned char As[2][NA][BM * 64];
    __shared__ __attribute__((aligned(16))) unsigned char Bs[2][NB][BN * 64];
    __shared__ float2 s_stat[OWN ? BM : 1];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = bx * BM, n0 = by * BN;
    // a thread moves the piece tid % 8 of the rows tid / 8 + 32 i of a chunk.  (Rows beyond the last token or feature hold the first one: they
    // reach no output but their own, which is not stored)
    const int pc = tid & 7, prow = tid >> 3;
    const T *ap[2], *bp[BP ? 1 : 2 * WN];
    float mean[2], rstd[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = t0 + prow + 32 * i;
        const int tc = t < g.tokens ? t : 0;
        if constexpr (PROJ) {
            const int rl = tc / g.L, l = tc - rl * g.L;
            ap[i] = (const T*)g.a + ((int64_t)(g.r0 + rl) * g.sr + (int64_t)l * g.sl) * g.K;
            if constexpr (OWN) {         // (the eight lanes of a row, as in token_row)
                constexpr bool V = VEC != 0;
                float4 r1[1], r2[2], r4[4], r8[8];
                if (g.K <= 32) row_stats<T, V, 1>(ap[i], g.K, pc, g.eps, mean[i], rstd[i], r1);
                else if (g.K <= 64) row_stats<T, V, 2>(ap[i], g.K, pc, g.eps, mean[i], rstd[i], r2);
                else if (g.K <= 128) row_stats<T, V, 4>(ap[i], g.K, pc, g.eps, mean[i], rstd[i], r4);
                else if (g.K <= 256) row_stats<T, V, 8>(ap[i], g.K, pc, g.eps, mean[i], rstd[i], r8);
                else row_stats<T, V, 0>(ap[i], g.K, pc, g.eps, mean[i], rstd[i], r1);
                if (pc == 0) s_stat[prow + 32 * i] = make_float2(mean[i], rstd[i]);
            } else {
                const float2 st = *reinterpret_cast<const float2*>(g.stats + 2 * (size_t)tc);
                mean[i] = st.x;
                rstd[i] = st.y;
            }
            rstd[i] *= kUp;
        } else {
            ap[i] = (const T*)g.a + (size_t)tc * g.K;
        }
    }
#pragma unroll
    for (int i = 0; i < (BP ? 0 : 2 * WN); ++i) {
        const int n = n0 + prow + 32 * i;
        const int nc = n < g.N ? n : 0;
        if constexpr (PROJ) {
            const int seg = nc / g.Hd;
            const void* w = seg == 0 ? g.w[0] : (seg == 1 ? g.w[1] : (seg == 2 ? g.w[2] : g.w[3]));
            bp[i] = (const T*)w + (size_t)(nc - seg * g.Hd) * g.K;
        } else {
            bp[i] = (const T*)g.w[0] + (size_t)nc * g.K;
        }
    }
    struct Chunk {
        Load a[2], b[BP ? 1 : 2 * WN], gm, bt;
    };
    const unsigned bs_lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)&Bs[0][0][0]);
    auto fetch = [&](Chunk& c, int k0) __attribute__((always_inline)) {
        const int k = k0 + 4 * pc;
#pragma unroll
        for (int i = 0; i < 2; ++i) c.a[i].fetch(ap[i], k, g.K);
#pragma unroll
        for (int i = 0; i < (BP ? 0 : 2 * WN); ++i) c.b[i].fetch(bp[i], k, g.K);
        if constexpr (PROJ) {
            c.gm.fetch((const T*)g.ln_g, k, g.K);
            c.bt.fetch((const T*)g.ln_b, k, g.K);
        }
    };
    // BP: the planes of a chunk, 3 WN KiB per wavefront (a block's rows of a plane are one piece of memory)
    const int np = plane_rows(g.N);
    const unsigned char* planes = BP ? g.planes + (size_t)n0 * 64 : nullptr;
    uint32_t plane_lane[BP ? 3 * WN : 1];
    if constexpr (BP) {
#pragma unroll
        for (int i = 0; i < 3 * WN; ++i) {
            const int c = 4 * i + wave, j = c / (4 * WN);
            plane_lane[i] = (uint32_t)(j * np * 64 + (c - j * 4 * WN) * 1024) + 16u * lane;
        }
    }
    auto fetch_planes = [&](int buf) __attribute__((always_inline)) {
        if constexpr (BP) {
#pragma unroll
            for (int i = 0; i < 3 * WN; ++i) load16_to_lds(planes, plane_lane[i], bs_lds + (unsigned)(buf * NB * BN * 64 + (4 * i + wave) * 1024));
            planes += (size_t)3 * np * 64;
        }
    };
    auto stash = [&](const Chunk& c, int buf, int k0) __attribute__((always_inline)) {
        const int k = k0 + 4 * pc;
        float4 gv, bv;
        if constexpr (PROJ) {
            gv = c.gm.value(k, g.K);
            bv = times4_piece<VEC != 0>(c.bt.value(k, g.K), kUp);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = prow + 32 * i;
            float4 v = c.a[i].value(k, g.K);
            if constexpr (!PROJ && NA == 3) v = times4_piece<VEC != 0>(v, kUp);
            if constexpr (PROJ)       // (beyond K gamma and beta are zero, and so is the result)
                v = make_float4((v.x - mean[i]) * rstd[i] * gv.x + bv.x, (v.y - mean[i]) * rstd[i] * gv.y + bv.y,
                                (v.z - mean[i]) * rstd[i] * gv.z + bv.z, (v.w - mean[i]) * rstd[i] * gv.w + bv.w);
            const Planes<NA> sp = split4<NA>(v);
#pragma unroll
            for (int j = 0; j < NA; ++j) *reinterpret_cast<uint2*>(&As[buf][j][row * 64 + piece_place(row, pc)]) = sp.p[j];
        }
#pragma unroll
        for (int i = 0; i < (BP ? 0 : 2 * WN); ++i) {
            const int row = prow + 32 * i;
            const float4 v = c.b[i].value(k, g.K);
            const Planes<NB> sp = split4<NB>(NB == 3 ? times4_piece<VEC != 0>(v, kUp) : v);
#pragma unroll
            for (int j = 0; j < NB; ++j) *reinterpret_cast<uint2*>(&Bs[buf][j][row * 64 + piece_place(row, pc)]) = sp.p[j];
        }
    };
    f32x16 acc[WN], low[WN];
#pragma unroll
    for (int n = 0; n < WN; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = low[n][v] = 0.f;
    const int wt = wave >> 1, wn = WN * (wave & 1);
    // A chunk's operands are requested two chunks ahead (a chunk's matrix instructions are over before memory answers), its planes, from L2, one; while
    // a chunk is contracted the next one is split and stored.
    const int last = (g.K - 1) & ~31;
    auto round = [&](Chunk& c1, Chunk& c2, int buf, int k0, auto ahead_c) __attribute__((always_inline)) {       // c1: chunk k0 + 32, c2: the one behind it, as far as there are any
        constexpr int ahead = decltype(ahead_c)::value;
        if constexpr (ahead > 0) fetch_planes(buf ^ 1);
        if constexpr (ahead > 1) fetch(c2, k0 + 64 < last ? k0 + 64 : last);              // (past the end: a harmless repeat, so that no load is under a condition)
        __builtin_amdgcn_sched_barrier(0);
        Frag av[2][NA], bv[2][WN][NB];
        const int sw = (col >> 2) & 3;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int at = col * 64 + (((2 * i + hf) ^ sw) & 3) * 16;            // (rows 32 apart: the same places)
#pragma unroll
            for (int j = 0; j < NA; ++j) av[i][j].u = *reinterpret_cast<const uint4*>(&As[buf][j][32 * wt * 64 + at]);
#pragma unroll
            for (int n = 0; n < WN; ++n) {
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[i][n][j].u = *reinterpret_cast<const uint4*>(&Bs[buf][j][32 * (wn + n) * 64 + at]);
                mfma_split<NA, NB>(av[i], bv[i][n], acc[n], low[n]);
            }
        }
        if constexpr (ahead > 0) {
            stash(c1, buf ^ 1, k0 + 32);              // (read last in the round before, and that round's barrier has passed)
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (BP) __builtin_amdgcn_s_waitcnt(ahead > 1 ? (PROJ ? 0x0F74 : 0x0F72) : kWaitVmcnt0);      // vmcnt: all but c2's four (two) loads
            __syncthreads();
        }
    };
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 0> none{};
    Chunk cur, nxt;
    fetch_planes(0);
    fetch(cur, 0);
    fetch(nxt, last < 32 ? last : 32);
    __builtin_amdgcn_sched_barrier(0);
    stash(cur, 0, 0);
    if constexpr (BP) __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    int k0 = 0;
    for (; k0 + 64 < g.K; k0 += 64) {
        round(nxt, cur, 0, k0, two);
        round(cur, nxt, 1, k0 + 32, two);
    }
    if (k0 + 32 < g.K) {
        round(nxt, cur, 0, k0, one);
        round(cur, nxt, 1, k0 + 32, none);
    } else {
        round(nxt, cur, 0, k0, none);
    }
#pragma unroll
    for (int n = 0; n < WN; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = (acc[n][v] + low[n][v]) * down;
    // lane = feature, register v = token 8 (v / 4) + 4 hf + v % 4 of the wavefront's 32: 128-byte runs per token.  FULL: all
    // of its tokens exist (the checks are branches around every store otherwise)
    const int tw = t0 + 32 * wt;
    if (tw >= g.tokens) return;                                  // (no barrier after this point)
    // An operand that is infinite, or rounds to infinity, leaves NaN in its planes' products, and sums near the top of the range may overflow in a part: any
    // result that is not finite is formed again (float32_tile)
    float zero = 0.f;                   // (stays so while everything is finite)
#pragma unroll
    for (int n = 0; n < WN; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) zero = fmaf(acc[n][v], 0.f, zero);
    if (__builtin_expect(__ballot(zero != 0.f) != 0, 0)) {
#pragma unroll
        for (int n = 0; n < WN; ++n)
            float32_tile<T, PROJ, VEC != 0>(g, tw, n0 + 32 * (wn + n), OWN ? s_stat + 32 * wt : nullptr, acc[n]);
    }
    auto emit = [&](auto full_c) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full_c)::value;
        // element offset of token tw + x in out: one division per wavefront where a row of tokens is at least a tile long
        const int rl0 = tw / g.L, l0 = tw - rl0 * g.L;
        auto token_at = [&](int x) __attribute__((always_inline)) -> int64_t {
            int l = l0 + x, r = rl0;
            if (g.L >= 32) {
                const bool wrap = l >= g.L;
                l -= wrap ? g.L : 0;
                r += wrap;
            } else {
                r = (tw + x) / g.L;
                l = tw + x - r * g.L;
            }
            return ((int64_t)(g.r0 + r) * g.sr + (int64_t)l * g.sl) * g.N;
        };
#pragma unroll
        for (int n = 0; n < WN; ++n) {
            const int f = n0 + 32 * (wn + n) + col;
            if (f >= g.N) continue;
            if constexpr (PROJ) {
                const int seg = f / g.Hd;
                if (seg == 3) {
                    const float bias = to_f32<T>(((const T*)g.bvec)[f - 3 * g.Hd]);
                    float top = 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        acc[n][v] = 1.f + __expf(-(acc[n][v] + bias));
                        top = fmaxf(top, acc[n][v]);
                    }
                    if (__ballot(top >= 0x1p126f)) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[n][v] = 1.f / acc[n][v];
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[n][v] = reciprocal(acc[n][v]);
                    }
                } else {
                    const float scale = seg == 0 ? g.qscale : 1.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[n][v] *= scale;
                }
                // (a uniform address that moves on by a token and an offset per lane: nothing for the vector unit to add)
                char* dst = (char*)g.cdst + (size_t)tw * g.N * sizeof(T);
                const uint32_t lane_at = (uint32_t)(f + 4 * hf * g.N) * sizeof(T);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int x = 8 * (v >> 2) + (v & 3);
                    if (FULL || tw + x + 4 * hf < g.tokens) *reinterpret_cast<T*>(dst + lane_at) = from_f32<T>(acc[n][v]);
                    dst += (size_t)((v & 3) == 3 ? 5 : 1) * g.N * sizeof(T);
                }
            } else {
                const float bias = to_f32<T>(((const T*)g.bvec)[f]);
                float add[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) add[v] = 0.f;
                if (g.res) {          // (the thread that stores an element is the one that read it: in place is safe)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int x = 8 * (v >> 2) + 4 * hf + (v & 3);
                        if (FULL || tw + x < g.tokens) add[v] = to_f32<T>(((const T*)g.res)[token_at(x) + f]);
                    }
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int x = 8 * (v >> 2) + 4 * hf + (v & 3);
                    if (FULL || tw + x < g.tokens) ((T*)g.cdst)[token_at(x) + f] = from_f32<T>(acc[n][v] + bias + add[v]);
                }
            }
        }
    };
    if (tw + 32 <= g.tokens) emit(std::integral_constant<bool, true>{});
    else emit(std::integral_constant<bool, false>{});
}

template <typename T, bool PROJ, int VEC, int WN, bool BP>
__global__ __launch_bounds__(256, WN == 1 ? (sizeof(T) == 2 ? 4 : 3) : 2) void k_gemm_generic(GenericGemmArgs g) {
    gemm_block<T, PROJ, VEC, WN, BP, false>(g, blockIdx.x, blockIdx.y);
}
// The projections of a small call and, in the blocks behind theirs, the pair bias, on which they do not depend (one_launch).
template <typename T, int VEC>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 4 : 3) void k_proj_rows_generic(GenericGemmArgs g, RowsArgs a, int nx, int gemm_blocks, int pair_vec) {
    if ((int)blockIdx.x < gemm_blocks) {
        const int by = (int)blockIdx.x / nx;
        gemm_block<T, true, VEC, 1, false, true>(g, (int)blockIdx.x - by * nx, by);
    } else if (pair_vec) {
        pair_rows<T, true>(a, (int)blockIdx.x - gemm_blocks);
    } else {
        pair_rows<T, false>(a, (int)blockIdx.x - gemm_blocks);
    }
}

// ---------------------------------------------------------------------------------------
// Attention: a wavefront per 32 queries of one (batch row, head), up to eight of them in a block, which shares the keys
// and values of that (row, head) through LDS, `keys` of them at a time (all of them for lengths up to 160 at d = 32:
// then every load of the block is in flight together and two barriers are all it needs).  S^T = K Q^T puts a query
// in a lane: maximum and sum are lane-local but for one exchange between the halves, and registers 8 c .. 8 c + 7 of the
// exponentiated tile, split into planes, are the B operand of step c of O^T = V^T P^T as they stand (the keys 16 c + 8 i + 4 hf + e). The bias is added to the finished products (as the
// accumulator's starting value it was rounded with every one of them), the key mask (0 or -inf) selects, in tiles that hold a masked key.  Online softmax; a query without
// any unmasked key gets zero context.  Output o = gate * context.
// Bound by the vector unit (exponentials, the planes of P: 260 instructions per 32 x 32 tile against 24 matrix instructions of 32 cycles).  Up to 32 channels it is held
// to 128 registers: with 155 a second block of five wavefronts did not fit a compute unit (64 x 155 tokens: 31 us instead of 25, both under the profiler); with bfloat16
// storage, whose operands are one plane, to 96: with 112 the same call at 16 heads of 8 channels, all launches, 65.6 us instead of 57.4.
// Weights below 2^-126 of the largest are zeros here and those below 2^-109 lose bits; whether any counts is decided once per query behind the loops (the smallest score
// and the context tell): exponentials with a way of their own for tiles that hold any take 0.6 % more of a call, over 240 shapes, than the smallest score.
struct GenericAttnArgs {
    const void* qkvg;
    const float* bias;       // [H][L][Lb] or NULL
    const float* mask;
    int64_t sr, sl;
    int r0, rows, L, Lb, H, d, keys;
    void* o;
};

// LDS per key: the planes of k (a row of channels per key, padded to an odd number of 16-byte pieces), of v^T and the mask term; per channel of v^T a
// pad of 16 bytes, which makes the pitch of its rows an odd number of pieces.
template <typename T>
constexpr int attn_planes() { return sizeof(T) == 4 ? 3 : 1; }
template <int DG>
constexpr int attn_k_pitch() { return DG == 1 ? 16 : 16 * DG + 16; }
template <typename T, int DG>
constexpr size_t attn_smem_bytes(int keys) {
    return (size_t)keys * (attn_planes<T>() * (attn_k_pitch<DG>() + 16 * DG) + 4) + attn_planes<T>() * 8 * DG * 16;
}

// the lane's index formed anew: what comes behind the loops holds no registers through them
__device__ __forceinline__ int fresh_lane() {
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}
// The context and (partial, per half-wave) sum of the wavefront's queries with `again`, all products on the float32 instruction: the operands come from the
// projected tensors, a lane's key, query or channel row.  Register v of the exponentiated tile is the B operand of instruction v of O^T = V^T P^T
// (its halves hold the keys 8 (v / 4) + v % 4 and that + 4).  Per 32 channels anew, for the registers; there are few such queries.
template <typename T, bool VEC, int DG>
__device__ __forceinline__ void float32_queries(const GenericAttnArgs& a, const T* base, const float* bias, const float* mask_row, int q0, bool again,
                                                f32x16 (&acc)[(8 * DG + 31) / 32], float& sum) {
    constexpr int NE = (8 * DG + 31) / 32;
    const int lane = fresh_lane(), col = lane & 31, hf = lane >> 5, Hd = a.H * a.d, N4 = 4 * Hd;
    const int qc = q0 + col < a.L ? q0 + col : a.L - 1;
    const T *qrow = base + (size_t)qc * N4, *kb = base + Hd, *vb = kb + Hd;
    const float* brow = bias ? bias + (size_t)qc * a.Lb : nullptr;
    float l = 0.f;
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        if (32 * n >= a.d) break;
        const int ch = 32 * n + col < a.d ? 32 * n + col : a.d - 1;
        f32x16 c;
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = 0.f;
        float m = -INFINITY;
        l = 0.f;
#pragma unroll 1
        for (int kt = 0; kt < a.L; kt += 32) {
            const T* krow = kb + (size_t)(kt + col < a.L ? kt + col : a.L - 1) * N4;
            f32x16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll 1
            for (int e0 = 0; e0 < a.d; e0 += 8) {
                const float4 kf = load4<T, VEC>(krow, e0 + 4 * hf, a.d), qf = load4<T, VEC>(qrow, e0 + 4 * hf, a.d);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.x, qf.x, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.y, qf.y, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.z, qf.z, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.w, qf.w, s, 0, 0, 0);
            }
            uint32_t live = 0;
            int k0 = kt + 4 * hf;
            asm volatile("" : "+v"(k0));           // (opaque: the addresses of all keys are formed here, none is held through the loop)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = k0 + 8 * (v >> 2) + (v & 3);
                const bool ok = k < a.L && (!mask_row || mask_row[(int64_t)k * a.sl] != 0.f);
                live |= ok ? 1u << v : 0u;
                s[v] = ok ? s[v] + (brow ? brow[k] : 0.f) : -INFINITY;
            }
            float tmax = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
            const float m_new = fmaxf(m, fmaxf(tmax, other_half(tmax))), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2f(m - ref);
            m = m_new;
            float part = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = exp2f(s[v] - ref);
                part += s[v];
            }
            l = l * alpha + part;
            f32x16 pv;
#pragma unroll
            for (int v = 0; v < 16; ++v) pv[v] = 0.f;
            asm volatile("" : "+v"(k0));
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = k0 + 8 * (v >> 2) + (v & 3);
                const float x = (live >> v) & 1 ? to_f32<T>(vb[(size_t)k * N4 + ch]) : 0.f;
                pv = __builtin_amdgcn_mfma_f32_32x32x2f32(x, s[v], pv, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) c[v] = fmaf(c[v], alpha, pv[v]);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = again ? c[v] : acc[n][v];
    }
    sum = again ? l : sum;
}

// Whether weights below 2^-109 may count in the lane's context: a channel of it is below 2^-80 times the largest of that channel's values.
template <typename T, bool VEC, int DG>
__device__ __forceinline__ bool small_weights_count(const GenericAttnArgs& a, const T* base, const float* mask_row, const f32x16 (&acc)[(8 * DG + 31) / 32], float sum) {
    constexpr int NG = DG < 4 ? DG : 4;              // pieces of a lane per 32 channels
    const int lane = fresh_lane(), col = lane & 31, hf = lane >> 5, Hd = a.H * a.d;
    bool low = false;
#pragma unroll
    for (int n = 0; n < (8 * DG + 31) / 32; ++n) {
        float top[4 * NG];
#pragma unroll
        for (int i = 0; i < 4 * NG; ++i) top[i] = 0.f;
#pragma unroll 1
        for (int k = col; k < a.L; k += 32) {
            if (mask_row && mask_row[(int64_t)k * a.sl] == 0.f) continue;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const float4 v = load4<T, VEC>(base + (size_t)k * 4 * Hd + 2 * Hd, 32 * n + 8 * g + 4 * hf, a.d);
                top[4 * g] = fmaxf(top[4 * g], fabsf(v.x));
                top[4 * g + 1] = fmaxf(top[4 * g + 1], fabsf(v.y));
                top[4 * g + 2] = fmaxf(top[4 * g + 2], fabsf(v.z));
                top[4 * g + 3] = fmaxf(top[4 * g + 3], fabsf(v.w));
            }
        }
#pragma unroll 1
        for (int o = 16; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < 4 * NG; ++i) top[i] = fmaxf(top[i], __shfl_xor(top[i], o, 64));
#pragma unroll
        for (int i = 0; i < 4 * NG; ++i) low = low || fabsf(acc[n][i]) < top[i] * 0x1p-80f;
    }
    return low && half_sum(sum) > 0.f;
}

template <typename T, bool VEC, int DG>      // DG: head dimension in groups of 8 channels (rounded up)
__global__ __launch_bounds__(512, DG <= 4 ? (sizeof(T) == 2 && (VEC || DG < 4) ? 5 : 4) : 2) void k_attn_generic(GenericAttnArgs a) {
    constexpr int DP = 8 * DG, NP = attn_planes<T>(), KP = attn_k_pitch<DG>(), NE = (DP + 31) / 32, NS = (DP + 15) / 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int VP = 2 * a.keys + 16;                                   // bytes of a row of v^T
    unsigned char* s_k = smem;                                        // [NP][keys][KP]
    unsigned char* s_v = s_k + (size_t)NP * a.keys * KP;              // [NP][DP][VP]
    float* s_m = reinterpret_cast<float*>(s_v + (size_t)NP * DP * VP);   // [keys] 0 or -inf
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5, nthreads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rl = blockIdx.x / a.H, h = blockIdx.x - rl * a.H;
    const int q0 = (blockIdx.y * (nthreads >> 6) + wave) * 32, qi = q0 + col;
    const bool active = q0 < a.L;
    const int qc = qi < a.L ? qi : a.L - 1;
    const int Hd = a.H * a.d, N4 = 4 * Hd;
    const T* base = (const T*)a.qkvg + (size_t)rl * a.L * N4 + (size_t)h * a.d;

    Frag qf[NS][NP];                                 // channels 16 s + 8 hf .. + 7 of the lane's query
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = 16 * s + 8 * hf + 4 * i;
            const float4 q = load4<T, VEC>(base + (size_t)qc * N4, e, a.d);
            const Planes<NP> sp = split4<NP>(NP == 3 ? times4(q, kUp) : q);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                qf[s][j].w[2 * i] = sp.p[j].x;
                qf[s][j].w[2 * i + 1] = sp.p[j].y;
            }
        }
    const float* brow = a.bias ? a.bias + ((size_t)h * a.L + qc) * a.Lb : nullptr;
    const float* mask_row = a.mask ? a.mask + (int64_t)(a.r0 + rl) * a.sr : nullptr;
    f32x16 acc[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    float m = -INFINITY, sum = 0.f;                  // m: reference of the exponentials
    float smin = INFINITY;                           // smallest score, those of masked keys among them

    for (int c0 = 0; c0 < a.L; c0 += a.keys) {
        const int nk = a.L - c0 < a.keys ? a.L - c0 : a.keys, nkp = (nk + 31) & ~31;
        if (c0) __syncthreads();                     // every wavefront is done with the keys before
        for (int k = tid; k < nkp; k += nthreads) {
            bool ok = k < nk;
            if (ok && mask_row) ok = mask_row[(int64_t)(c0 + k) * a.sl] != 0.f;
            s_m[k] = ok ? 0.f : -INFINITY;
        }
        // k: pieces of four channels of a key.  v^T: four neighbouring keys of a channel, lanes along the channels; the keys 16 c + 8 i + 4 hf + e of a
        // row lie in the places 16 c + 8 hf + 4 i + e, so that those of a half-wave of P^T, see below, are one piece.  As many of both, and U
        // of each are on their way together (a wavefront per 32 keys: all that the block needs, up to 32 channels).
        constexpr int PR = DP / 4, U = DG < 4 ? DG : 4;
        const T *kb = base + (size_t)c0 * N4 + Hd, *vb = kb + Hd;
        for (int b0 = 0; b0 < nkp * PR; b0 += U * nthreads) {
            Piece<T, VEC> kp[U];
            T vv[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int id = b0 + u * nthreads + tid, k = id / PR, k4 = 4 * (id / DP), e = id % DP;
                kp[u].fetch(kb + (size_t)(k < nk ? k : nk - 1) * N4, 4 * (id % PR), a.d);
#pragma unroll
                for (int i = 0; i < 4; ++i) vv[u][i] = vb[(size_t)(k4 + i < nk ? k4 + i : nk - 1) * N4 + (e < a.d ? e : a.d - 1)];
            }
            if (b0 == 0) __syncthreads();         // the mask terms are there
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int id = b0 + u * nthreads + tid, k = id / PR, k4 = 4 * (id / DP), e = id % DP;
                if (id >= nkp * PR) break;
                float4 kv = kp[u].value(4 * (id % PR), a.d);
                if constexpr (NP == 3) kv = times4_piece<VEC>(kv, kUp);
                const Planes<NP> ks = split4<NP>(keep4(k < nk, kv));
                const float4 m4 = *reinterpret_cast<const float4*>(s_m + k4);
                // (what a masked token holds may be anything, and 0 x NaN is NaN)
                const bool in = e < a.d;
                const float4 v4 = make_float4(in && m4.x == 0.f ? to_f32<T>(vv[u][0]) : 0.f, in && m4.y == 0.f ? to_f32<T>(vv[u][1]) : 0.f,
                                              in && m4.z == 0.f ? to_f32<T>(vv[u][2]) : 0.f, in && m4.w == 0.f ? to_f32<T>(vv[u][3]) : 0.f);
                const Planes<NP> vs = split4<NP>(NP == 3 ? times4(v4, kUp) : v4);
                const int at = (k4 & ~15) + 2 * (k4 & 4) + ((k4 & 8) >> 1);
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    *reinterpret_cast<uint2*>(s_k + (j * a.keys + k) * KP + 8 * (id % PR)) = ks.p[j];
                    *reinterpret_cast<uint2*>(s_v + (j * DP + e) * VP + 2 * at) = vs.p[j];
                }
            }
        }
        __syncthreads();
        if (!active) continue;
        for (int kt = 0; kt < nkp; kt += 32) {
            // lane = query, register 4 g + e = key kt + 8 g + 4 hf + e
            f32x16 s, lo;
            float4 bias[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) bias[g] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (brow) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {        // (beyond the row: any of it, those keys are masked)
                    const int k = c0 + kt + 8 * g + 4 * hf;
                    bias[g] = *reinterpret_cast<const float4*>(brow + (k < a.Lb ? k : a.Lb - 4));
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = lo[v] = 0.f;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                Frag kf[NP];
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    kf[j].u = *reinterpret_cast<const uint4*>(s_k + (j * a.keys + kt + col) * KP + (DG == 1 ? 0 : 32 * i + 16 * hf));
                    if (DG == 1 && hf) kf[j].u = make_uint4(0, 0, 0, 0);
                }
                mfma_split<NP, NP>(kf, qf[i], s, lo);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                constexpr float down = NP == 3 ? kDown * kDown : 1.f;
                s[4 * g] = fmaf(s[4 * g] + lo[4 * g], down, bias[g].x);
                s[4 * g + 1] = fmaf(s[4 * g + 1] + lo[4 * g + 1], down, bias[g].y);
                s[4 * g + 2] = fmaf(s[4 * g + 2] + lo[4 * g + 2], down, bias[g].z);
                s[4 * g + 3] = fmaf(s[4 * g + 3] + lo[4 * g + 3], down, bias[g].w);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) smin = fminf(smin, s[v]);
            if (__ballot(s_m[kt + col] != 0.f)) {                // (tiles with masked keys only)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 m4 = *reinterpret_cast<const float4*>(s_m + kt + 8 * g + 4 * hf);
                    // (a select, not a sum: what a masked key or the padded end of a bias row holds may be anything)
                    s[4 * g] = m4.x == 0.f ? s[4 * g] : m4.x;
                    s[4 * g + 1] = m4.y == 0.f ? s[4 * g + 1] : m4.y;
                    s[4 * g + 2] = m4.z == 0.f ? s[4 * g + 2] : m4.z;
                    s[4 * g + 3] = m4.w == 0.f ? s[4 * g + 3] : m4.w;
                }
            }
            float tmax = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
            tmax = fmaxf(tmax, other_half(tmax));
            // the reference follows the maximum only where a score exceeds it by more than 8: weights stay below 2^8, and most tiles rescale nothing
            if (__ballot(tmax > m + 8.f)) {
                const float m_new = fmaxf(m, tmax);
                const float alpha = exp2f(m - (m_new == -INFINITY ? 0.f : m_new));
                m = m_new;
                sum *= alpha;
#pragma unroll
                for (int n = 0; n < NE; ++n)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[n][v] *= alpha;
            }
            const float ref = m == -INFINITY ? 0.f : m;
            float part = 0.f;
            Frag pf[2][3];                           // step c of P^T: registers 8 c .. 8 c + 7, keys kt + 16 c + 8 i + 4 hf + e
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float4 p;
                p.x = __builtin_amdgcn_exp2f(s[4 * g] - ref);
                p.y = __builtin_amdgcn_exp2f(s[4 * g + 1] - ref);
                p.z = __builtin_amdgcn_exp2f(s[4 * g + 2] - ref);
                p.w = __builtin_amdgcn_exp2f(s[4 * g + 3] - ref);
                part += p.x;
                part += p.y;
                part += p.z;
                part += p.w;
                const Planes<3> sp = split4<3>(p);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    pf[g >> 1][j].w[2 * (g & 1)] = sp.p[j].x;
                    pf[g >> 1][j].w[2 * (g & 1) + 1] = sp.p[j].y;
                }
            }
            sum += part;
            // the tile's own sums, so that a few products and the tiles round, not all keys in a row.  lane = query, register v = channel
            // 32 n + 8 (v / 4) + 4 hf + v % 4; channels beyond DP read a row again and are dropped
#pragma unroll
            for (int n = 0; n < NE; ++n) {
                f32x16 pv, lv;
#pragma unroll
                for (int v = 0; v < 16; ++v) pv[v] = lv[v] = 0.f;
                const unsigned char* vr = s_v + (DP < 32 ? (col < DP ? col : 0) : 32 * n + col) * VP + 2 * kt + 16 * hf;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    Frag vf[NP];
#pragma unroll
                    for (int j = 0; j < NP; ++j) vf[j].u = *reinterpret_cast<const uint4*>(vr + j * DP * VP + 32 * c);
                    mfma_split<NP, 3>(vf, pf[c], pv, lv);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[n][v] += pv[v] + lv[v];
            }
        }
    }
    if (!active) return;
    if constexpr (NP == 3) {
#pragma unroll
        for (int n = 0; n < NE; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] *= kDown;
    }
    // Contexts that are not finite, as in the projections (an infinite value against the lower planes of a weight, a product of huge and tiny factors, a
    // score of -infinity), and those that may owe something to a weight of which the exponential's instruction makes zero (below 2^-126) or whose last
    // plane loses bits (below 2^-109): the query again with float32 products and the library's exponential, from the projected tensors, its own
    // maximum in every tile.  The queries' results are their own; one that begins with a NaN, as all of a
    // token with anything that is not finite do, is left as it is.
    float zero = sum * 0.f;             // (stays so while everything is finite)
#pragma unroll
    for (int n = 0; n < NE; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) zero = fmaf(acc[n][v], 0.f, zero);
    bool odd = zero != 0.f;
    if (__builtin_expect(__ballot(smin < m - 100.f) != 0, 0)) odd = odd || small_weights_count<T, VEC, DG>(a, base, mask_row, acc, sum);
    const uint64_t b = __ballot(odd);
    if (__builtin_expect(b != 0, 0)) {
        const int ln = fresh_lane(), qn = q0 + (ln & 31) < a.L ? q0 + (ln & 31) : a.L - 1;
        const float first = to_f32<T>(base[(size_t)qn * N4]);
        const uint32_t again = ((uint32_t)b | (uint32_t)(b >> 32)) & ~(uint32_t)__ballot(first != first);
        if (again) float32_queries<T, VEC, DG>(a, base, a.bias ? a.bias + (size_t)h * a.L * a.Lb : nullptr, mask_row, q0, (again >> (ln & 31)) & 1, acc, sum);
    }
    if (qi >= a.L) return;
    sum += other_half(sum);
    const float inv = sum > 0.f ? 1.f / sum : 0.f;
    T* op = (T*)a.o + ((size_t)rl * a.L + qi) * Hd + (size_t)h * a.d;
    const T* gp = base + (size_t)qi * N4 + 3 * Hd;
#pragma unroll
    for (int n = 0; n < NE; ++n)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e = 32 * n + 8 * g + 4 * hf;
            if (e >= a.d) continue;
            const float4 gt = load4<T, VEC>(gp, e, a.d);
            store4<T, VEC>(op, e, a.d, make_float4(acc[n][4 * g] * inv * gt.x, acc[n][4 * g + 1] * inv * gt.y,
                                                   acc[n][4 * g + 2] * inv * gt.z, acc[n][4 * g + 3] * inv * gt.w));
        }
}

// ---------------------------------------------------------------------------------------
static bool aligned_to(const void* p, size_t n) { return ((uintptr_t)p & (n - 1)) == 0; }

// Whether the merged projection's loads are whole 16-byte (bfloat16: 8-byte) pieces.
template <typename T>
static bool proj_vec(const Problem& p, const ff_attn_weights& w, const void* x) {
    const size_t al = 4 * sizeof(T);
    return p.c % 4 == 0 && aligned_to(x, al) && aligned_to(w.ln_g, al) && aligned_to(w.ln_b, al) && aligned_to(w.w_q, al) &&
           aligned_to(w.w_k, al) && aligned_to(w.w_v, al) && aligned_to(w.w_g, al);
}
// The place of the split projection weights, or NULL: the context's, which nobody needs before the attention, if a chunk has tokens enough for
// it to hold them (then the weights are also split often enough to be worth a pass of their own: each 64 tokens do it again otherwise).
template <typename T>
static unsigned char* weight_planes(const Problem& p, const ff_attn_weights& w, const void* x, const Workspace& ws) {
    if (sizeof(T) != 4 || p.c % 32 != 0 || !proj_vec<T>(p, w, x)) return nullptr;
    return (size_t)6 * plane_rows(4 * p.Hd) * p.c <= (size_t)ws.chunk * p.L * p.Hd * 4 ? (unsigned char*)ws.o : nullptr;
}

// Whether the projections form the token statistics themselves and the pair bias rides in their launch: where a chunk's projections are at most four
// blocks per compute unit and the pairs at most forty (their blocks hold the projections' LDS and registers).  The rows' launch and its latency are a fifth of a small call: 8 x 32
// row attention of 32 channels 18.0 -> 15.6 us, 46 x 46 triangle attention of 256 channels 40.7 -> 35.4 (40.3 with a limit of one block), 8 x 200 row attention 52.7 -> 46.8 (with at most four blocks of pairs 52.6),
// 4 x 256 of 32 channels 31.9 -> 29.9, 30 x 100 43.2 -> 40.6.  With eight blocks 53 x 100 60.8 -> 64, with sixteen 64 x 155 90 -> 107: every block of 64 features reads all of its tokens twice.
// Rows of more than 256 channels do not stay in registers, so a block reads its tokens twice more for their statistics: 114 x 56 column attention of 1600 channels 124
// us instead of 102, 64 x 155 row attention of 512 channels 105 instead of 84.  There the pair bias decides, a serial pass over H + 2 rows per pair, in triangle
// attention: with two heads or more and few blocks of few tokens it hides behind the projections (31 x 31 of 1511 channels, 15 heads, 398 us instead of 490, 78 x 78 of
// 320 channels, 4 heads, 49 instead of 56, 100 x 100 of 640 channels, 4 heads of 8, 80 instead of 90; 115 x 115 of it, above the line of tokens times blocks, 113
// instead of 102, and 128 x 128 of 1152 channels, 2 heads of 16, 156 instead of 130; 23 x 23 of 1408 channels, 2 heads, 64 instead of 70, 100 x 100 of 1600 channels,
// one head of 32, 163 instead of 142).  With bfloat16 storage, half the bytes, every call with a bias (4 x 20 of 512 channels 29 us instead of 32), but rows of no
// whole pieces only in triangle attention of up to three blocks per compute unit (60 x 60 of 515 channels, 4 heads, 123 instead of 163; 70 x 70 of 1531 channels, 12
// heads, 1182 instead of 1023).
static bool one_launch(const Problem& p, const Workspace& ws) {
    const int64_t cu = compute_units(), tokens = (int64_t)ws.chunk * p.L, features = (4 * p.Hd + 63) / 64, blocks = (tokens + 63) / 64 * features;
    if (blocks > 4 * cu || (p.has_bias && (int64_t)p.L * p.L > 40 * 32 * cu)) return false;
    if (p.c <= 256) return true;
    const bool triangle = p.mode == FF_TRI_START || p.mode == FF_TRI_END;
    if (p.dtype == FF_BF16) return p.has_bias && (p.c % 4 == 0 || (triangle && blocks <= 3 * cu));
    return triangle && p.H >= 2 && 2 * blocks <= (p.H > 2 ? 5 : 2) * cu && tokens * blocks <= 64 * cu * cu;
}

// the pair bias in `a`; returns whether its loads are whole pieces
template <typename T>
static bool pair_args(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, RowsArgs& a) {
    if (p.mode == FF_MSA_ROW) {
        a.src = z; a.sq = p.L; a.sk = 1; a.cp = p.c_z; a.g = w.lnz_g; a.b = w.lnz_b;
    } else {
        a.src = x; a.sq = p.sr; a.sk = p.sl; a.cp = p.c; a.g = w.ln_g; a.b = w.ln_b;
    }
    a.wb = w.w_b;
    a.pair_blocks = (int)(((int64_t)p.L * p.L + 31) / 32);
    return a.cp % 4 == 0 && aligned_to(a.src, 4 * sizeof(T)) && aligned_to(a.g, 4 * sizeof(T)) && aligned_to(a.b, 4 * sizeof(T)) &&
           aligned_to(a.wb, 4 * sizeof(T));
}
static RowsArgs rows_args(const Problem& p, const void* x, const Workspace& ws, int r0, int rows) {
    RowsArgs a{};
    a.H = p.H; a.L = p.L; a.Lb = bias_pitch(p.L); a.bias = ws.bias; a.eps = p.eps;
    a.x = x; a.sr = p.sr; a.sl = p.sl; a.c = p.c; a.r0 = r0; a.tokens = rows * p.L; a.stats = ws.stats;
    return a;
}

// token statistics of `rows` batch rows from r0 on, the pair bias if `pairs`, and the weights' planes
template <typename T>
static ff_status rows_t(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const Workspace& ws, int r0,
                        int rows, bool pairs, hipStream_t st) {
    if (one_launch(p, ws)) return FF_OK;
    RowsArgs a = rows_args(p, x, ws, r0, rows);
    bool vec = p.c % 4 == 0 && aligned_to(x, 4 * sizeof(T));
    if (pairs) vec = pair_args<T>(p, w, x, z, a) && vec;
    a.token_blocks = (a.tokens + 31) / 32;
    a.planes = weight_planes<T>(p, w, x, ws);
    int split_blocks = 0;
    if (a.planes) {
        a.w[0] = w.w_q; a.w[1] = w.w_k; a.w[2] = w.w_v; a.w[3] = w.w_g; a.Hd = p.Hd;
        split_blocks = (plane_rows(4 * p.Hd) * (p.c / 4) + 255) / 256;
    }
    const dim3 grid((unsigned)(a.pair_blocks + a.token_blocks + split_blocks));
    if (vec) hipLaunchKernelGGL((k_rows_generic<T, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_rows_generic<T, false>), grid, dim3(256), 0, st, a);
    return check_launch("rows (generic)");
}

template <typename T, bool PROJ, int VEC, bool BP>
static void launch_gemm_vec(const GenericGemmArgs& g, hipStream_t st) {
    // 128 features per block (the tokens are split half as often) where that gives at least four blocks per compute unit: with it from two blocks on
    // 128 x 40 tokens of 256 channels 54 us instead of 51, 200 x 200 tokens of 64 channels 83 instead of 78; from eight on 64 x 155 tokens 90 instead of 86;
    // never, 256 x 256 tokens 530 instead of 497.
    const unsigned nx = (unsigned)((g.tokens + 63) / 64);
    const unsigned wide = (unsigned)((g.N + 127) / 128);
    if ((int64_t)nx * wide >= 4 * compute_units())
        hipLaunchKernelGGL((k_gemm_generic<T, PROJ, VEC, 2, BP>), dim3(nx, wide), dim3(256), 0, st, g);
    else
        hipLaunchKernelGGL((k_gemm_generic<T, PROJ, VEC, 1, BP>), dim3(nx, (unsigned)((g.N + 63) / 64)), dim3(256), 0, st, g);
}
template <typename T, bool PROJ>
static void launch_gemm(const GenericGemmArgs& g, bool vec, hipStream_t st) {
    if constexpr (PROJ && sizeof(T) == 4) {
        if (g.planes) return launch_gemm_vec<T, PROJ, 2, true>(g, st);
    }
    if (vec && g.K % 32 == 0) launch_gemm_vec<T, PROJ, 2, false>(g, st);
    else if (vec) launch_gemm_vec<T, PROJ, 1, false>(g, st);
    else launch_gemm_vec<T, PROJ, 0, false>(g, st);
}

template <typename T, bool VEC, int DG>
static ff_status launch_attn(GenericAttnArgs a, hipStream_t st) {
    // as many keys at a time as 72 KiB hold (two blocks per compute unit), a multiple of 32
    const int lp = (a.L + 31) & ~31;
    int keys = 32;
    while (keys < lp && attn_smem_bytes<T, DG>(keys + 32) <= 72 * 1024) keys += 32;
    a.keys = keys;
    const size_t smem = attn_smem_bytes<T, DG>(keys);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_generic<T, VEC, DG>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 72 * 1024);
    if (attr != hipSuccess) return fail(FF_EHIP, "k_attn_generic: dynamic LDS limit: %s", hipGetErrorString(attr));
    const int tiles = lp / 32;
    const int groups = (tiles + 7) / 8, waves = (tiles + groups - 1) / groups;
    hipLaunchKernelGGL((k_attn_generic<T, VEC, DG>), dim3((unsigned)(a.rows * a.H), groups), dim3(64 * waves), smem, st, a);
    return FF_OK;
}

template <typename T>
static ff_status chunk_t(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const float* mask, const void* res,
                         void* out, const Workspace& ws, int r0, int rows, hipStream_t st) {
    const int tokens = rows * p.L;
    const size_t al = 4 * sizeof(T);
    GenericGemmArgs g{};
    g.a = x; g.sr = p.sr; g.sl = p.sl; g.L = p.L; g.r0 = r0; g.tokens = tokens;
    g.K = p.c; g.N = 4 * p.Hd; g.stats = ws.stats; g.ln_g = w.ln_g; g.ln_b = w.ln_b;
    g.w[0] = w.w_q; g.w[1] = w.w_k; g.w[2] = w.w_v; g.w[3] = w.w_g; g.bvec = w.b_g; g.Hd = p.Hd;
    g.qscale = kLog2e / sqrtf((float)p.d);
    g.cdst = ws.qkvg;
    if (one_launch(p, ws)) {
        g.eps = p.eps;
        RowsArgs a = rows_args(p, x, ws, r0, rows);
        const int pair_vec = r0 == 0 && p.has_bias && pair_args<T>(p, w, x, z, a);
        const int nx = (tokens + 63) / 64, blocks = nx * ((g.N + 63) / 64);
        const dim3 grid((unsigned)(blocks + a.pair_blocks));
        if (!proj_vec<T>(p, w, x)) hipLaunchKernelGGL((k_proj_rows_generic<T, 0>), grid, dim3(256), 0, st, g, a, nx, blocks, pair_vec);
        else if (g.K % 32 != 0) hipLaunchKernelGGL((k_proj_rows_generic<T, 1>), grid, dim3(256), 0, st, g, a, nx, blocks, pair_vec);
        else hipLaunchKernelGGL((k_proj_rows_generic<T, 2>), grid, dim3(256), 0, st, g, a, nx, blocks, pair_vec);
    } else {
        g.planes = weight_planes<T>(p, w, x, ws);
        launch_gemm<T, true>(g, proj_vec<T>(p, w, x), st);
    }

    GenericAttnArgs a{};
    a.qkvg = ws.qkvg; a.bias = ws.bias; a.mask = mask; a.sr = p.sr; a.sl = p.sl; a.r0 = r0; a.rows = rows; a.L = p.L;
    a.Lb = bias_pitch(p.L); a.H = p.H; a.d = p.d; a.o = ws.o;
    ff_status ls = FF_OK;
#define FF_GEN_ATTN(DG)                                        \
    do {                                                       \
        if (p.d % 4 == 0) ls = launch_attn<T, true, DG>(a, st); \
        else ls = launch_attn<T, false, DG>(a, st);            \
    } while (0)
    if (p.d <= 8) FF_GEN_ATTN(1);
    else if (p.d <= 16) FF_GEN_ATTN(2);
    else if (p.d <= 32) FF_GEN_ATTN(4);
    else if (p.d <= 64) FF_GEN_ATTN(8);
    else FF_GEN_ATTN(16);
#undef FF_GEN_ATTN
    if (ls != FF_OK) return ls;

    GenericGemmArgs o{};
    o.a = ws.o; o.sr = p.sr; o.sl = p.sl; o.L = p.L; o.r0 = r0; o.tokens = tokens;
    o.K = p.Hd; o.N = p.c; o.w[0] = w.w_o; o.bvec = w.b_o; o.Hd = p.Hd; o.cdst = out; o.res = res;
    launch_gemm<T, false>(o, p.Hd % 4 == 0 && aligned_to(w.w_o, al), st);
    return check_launch("attention chunk (generic)");
}

}  // namespace gen

size_t generic_workspace(const Problem& p, int chunk, Workspace* ws, void* base) {
    using namespace gen;
    const size_t esz = p.dtype == FF_F32 ? 4 : 2;
    const size_t tokens = (size_t)chunk * p.L;
    size_t off = 0;
    char* b = (char*)base;
    ws->bias = nullptr;
    if (p.has_bias) {
        ws->bias = (float*)(b + off);
        off += align256((size_t)p.H * p.L * bias_pitch(p.L) * 4);
    }
    ws->prep = nullptr;
    ws->stats = (float*)(b + off);
    off += align256(tokens * 2 * 4);
    ws->qkvg = b + off;
    off += align256(tokens * 4 * p.Hd * esz);
    ws->o = b + off;
    off += align256(tokens * p.Hd * esz);
    ws->total = off;
    ws->chunk = chunk;
    return off;
}

// before the chunks: the pair bias and, in the same launch, the token statistics of the first chunk
ff_status generic_prepare(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const Workspace& ws, hipStream_t stream) {
    if (gen::one_launch(p, ws)) return FF_OK;
    Timed t(KK_GENERIC, stream);
    const int rows = ws.chunk < p.R ? ws.chunk : p.R;
    return p.dtype == FF_F32 ? gen::rows_t<float>(p, w, x, z, ws, 0, rows, p.has_bias, stream)
                             : gen::rows_t<bf16_t>(p, w, x, z, ws, 0, rows, p.has_bias, stream);
}

ff_status generic_chunk(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const float* mask,
                        const void* res, void* out, const Workspace& ws, int r0, int rows, hipStream_t stream) {
    if (r0 > 0) {
        const ff_status st = p.dtype == FF_F32 ? gen::rows_t<float>(p, w, x, nullptr, ws, r0, rows, false, stream)
                                               : gen::rows_t<bf16_t>(p, w, x, nullptr, ws, r0, rows, false, stream);
        if (st != FF_OK) return st;
    }
    return p.dtype == FF_F32 ? gen::chunk_t<float>(p, w, x, z, mask, res, out, ws, r0, rows, stream)
                             : gen::chunk_t<bf16_t>(p, w, x, z, mask, res, out, ws, r0, rows, stream);
}

}  // namespace ff
