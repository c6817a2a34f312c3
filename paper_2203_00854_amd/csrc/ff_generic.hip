// Generic kernel family: every step of the gated attention in float32, for any shape and for both storage types.  It
// is the float32 path (no bfloat16 anywhere when T = float) and the fallback for bfloat16 shapes the bfloat16
// matrix-core family does not take.  Steps follow FastFold Section 2.1 (projections, scaled dot product, softmax,
// product with V, output linear), Section 2.3 (axes, pair bias) and Section 5.2 (softmax with the mask and bias
// addends fused in; gate = bias + sigmoid + product).
//
// All contractions run on the float32 matrix instruction v_mfma_f32_32x32x2_f32: the same float32 products and sums
// as the vector unit's multiply-add at twice its rate, and the operands are read once per 32 x 32 tile instead of
// once per few outputs.  Operand layouts (wave64): A (32 x 2): lane l holds row l%32, column l/32; B (2 x 32): lane l
// holds column l%32, row l/32; C/D (32 x 32): lane l holds column l%32, register v holds row 8*(v/4) + 4*(l/32) + v%4.
// Which contraction index a lane's half stands for is free as long as A and B agree, so a lane reads four
// consecutive elements k0 + 4*half .. + 3 at once and feeds four instructions with them.
// Measured (row attention, 64 x 155 tokens of 256 channels, 8 heads of 32, 8.1 GFLOP): 1.40 ms with vector
// multiply-adds, a wavefront per query and per pair, 0.116 ms so (projections 59 us, attention 30, output
// projection 20, rows 9; the matrix cores alone need 53); 8 x 32 tokens of 32 channels: 33.8 -> 17.7 us, all launches.
//
// Workspace layout of this family, per chunk of `rows` batch rows, token t = rl*L + l:
//   stats [tokens][2]   float32 mean, 1/std of LayerNorm
//   qkvg  [tokens][4*Hd] T : q (times log2(e)/sqrt(d)), k, v, sigmoid gate
//   o     [tokens][Hd]   T : gate * context
//   bias  [H][L][Lb]     float32, times log2(e); rows padded to a multiple of four (16-byte reads)
#include "ff_common.h"

#include <type_traits>

namespace ff {
namespace gen {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

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
};

__device__ __forceinline__ float sum8(float v) {
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    return v;
}

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

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_rows_generic(RowsArgs a) {
    const int j8 = threadIdx.x & 7, r32 = threadIdx.x >> 3;
    if ((int)blockIdx.x < a.pair_blocks) {
        const int64_t pair = (int64_t)blockIdx.x * 32 + r32;
        if (a.cp <= 32) pair_row<T, VEC, 1>(a, pair, j8);
        else if (a.cp <= 64) pair_row<T, VEC, 2>(a, pair, j8);
        else if (a.cp <= 128) pair_row<T, VEC, 4>(a, pair, j8);
        else if (a.cp <= 256) pair_row<T, VEC, 8>(a, pair, j8);
        else pair_row<T, VEC, 0>(a, pair, j8);
        return;
    }
    const int t = ((int)blockIdx.x - a.pair_blocks) * 32 + r32;
    if (a.c <= 32) token_row<T, VEC, 1>(a, t, j8);
    else if (a.c <= 64) token_row<T, VEC, 2>(a, t, j8);
    else if (a.c <= 128) token_row<T, VEC, 4>(a, t, j8);
    else if (a.c <= 256) token_row<T, VEC, 8>(a, t, j8);
    else token_row<T, VEC, 0>(a, t, j8);
}

// ---------------------------------------------------------------------------------------
// GEMM, 32 WM tokens x 64 features per block of four wavefronts, contraction in chunks of 32 through double-buffered
// LDS (the next chunk travels to registers meanwhile).  WM = 4: a wavefront takes 32 tokens x 64 features; WM = 2:
// 32 x 32, twice the blocks, for launches that would otherwise leave compute units idle.
//   PROJ = true : A = LayerNorm(x) on the fly (stats, gamma, beta), B rows from w_q|w_k|w_v|w_g,
//                 epilogue: q scaled, gate = sigmoid(acc + b_g); C -> qkvg[t][4Hd]
//   PROJ = false: A = o[t][Hd], B = w_o, epilogue + b_o, C -> out at the token's address.
// Bound by the matrix cores: 64 cycles per instruction of 4096 flop (153 TFLOP/s for a large float32 product on this
// chip), against one 16-byte LDS read per operand and four instructions.
struct GenericGemmArgs {
    const void* a;         // x (PROJ) or o
    int64_t sr, sl;        // token strides of x / out
    int L, r0, tokens;     // chunk geometry
    int K, N;              // contraction length, output features
    const float* stats;
    const void *ln_g, *ln_b;
    const void* w[4];      // PROJ: w_q, w_k, w_v, w_g ([Hd][K] each); else w[0] = w_o [N][K]
    const void* bvec;      // PROJ: b_g [Hd]; else b_o [N]
    int Hd;
    float qscale;
    void* cdst;            // qkvg or out
    const void* res;       // !PROJ: residual added to the output (laid out like out, may be out itself) or NULL
};

template <typename T, bool PROJ, bool VEC, int WM>
__global__ __launch_bounds__(256) void k_gemm_generic(GenericGemmArgs g) {
    constexpr int BM = 32 * WM, NT = WM == 4 ? 2 : 1;          // tokens per block; 32-feature tiles per wavefront
    // rows of 32 floats, 16-byte piece p of row r in place p ^ (r & 7): conflict-free reads with lane = row
    __shared__ __attribute__((aligned(16))) float As[2][BM * 32];
    __shared__ __attribute__((aligned(16))) float Bs[2][64 * 32];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * BM, n0 = blockIdx.y * 64;
    // a thread moves the piece tid % 8 of the rows tid / 8 + 32 i of a chunk
    const int pc = tid & 7, prow = tid >> 3;
    const T *ap[WM], *bp[2];
    float mean[WM], rstd[WM];
    bool aok[WM], bok[2];
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int t = t0 + prow + 32 * i;
        aok[i] = t < g.tokens;
        const int tc = aok[i] ? t : 0;
        if constexpr (PROJ) {
            const int rl = tc / g.L, l = tc - rl * g.L;
            ap[i] = (const T*)g.a + ((int64_t)(g.r0 + rl) * g.sr + (int64_t)l * g.sl) * g.K;
            const float2 st = *reinterpret_cast<const float2*>(g.stats + 2 * (size_t)tc);
            mean[i] = st.x;
            rstd[i] = st.y;
        } else {
            ap[i] = (const T*)g.a + (size_t)tc * g.K;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = n0 + prow + 32 * i;
        bok[i] = n < g.N;
        const int nc = bok[i] ? n : 0;
        if constexpr (PROJ) {
            const int seg = nc / g.Hd;
            const void* w = seg == 0 ? g.w[0] : (seg == 1 ? g.w[1] : (seg == 2 ? g.w[2] : g.w[3]));
            bp[i] = (const T*)w + (size_t)(nc - seg * g.Hd) * g.K;
        } else {
            bp[i] = (const T*)g.w[0] + (size_t)nc * g.K;
        }
    }
    Piece<T, VEC> ra[WM], rb[2], gm, bt;
    auto fetch = [&](int k0) {
        const int k = k0 + 4 * pc;
#pragma unroll
        for (int i = 0; i < WM; ++i) ra[i].fetch(ap[i], k, g.K);
#pragma unroll
        for (int i = 0; i < 2; ++i) rb[i].fetch(bp[i], k, g.K);
        if constexpr (PROJ) {
            gm.fetch((const T*)g.ln_g, k, g.K);
            bt.fetch((const T*)g.ln_b, k, g.K);
        }
    };
    auto stash = [&](int buf, int k0) {
        const int k = k0 + 4 * pc;
        float4 gv, bv;
        if constexpr (PROJ) {
            gv = gm.value(k, g.K);
            bv = bt.value(k, g.K);
        }
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int row = prow + 32 * i;
            float4 v = ra[i].value(k, g.K);
            if constexpr (PROJ)       // (beyond K gamma and beta are zero, and so is the result)
                v = make_float4((v.x - mean[i]) * rstd[i] * gv.x + bv.x, (v.y - mean[i]) * rstd[i] * gv.y + bv.y,
                                (v.z - mean[i]) * rstd[i] * gv.z + bv.z, (v.w - mean[i]) * rstd[i] * gv.w + bv.w);
            *reinterpret_cast<float4*>(&As[buf][row * 32 + ((pc ^ (row & 7)) << 2)]) = keep4(aok[i], v);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = prow + 32 * i;
            *reinterpret_cast<float4*>(&Bs[buf][row * 32 + ((pc ^ (row & 7)) << 2)]) = keep4(bok[i], rb[i].value(k, g.K));
        }
    };
    // two sums per output, of the even and of the odd ones of every four contraction steps, added at the end: half as many roundings
    // in a row, none of which costs the matrix core anything
    f32x16 acc[NT], odd[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = odd[n][v] = 0.f;
    const int wt = WM == 4 ? wave : wave >> 1, wn = WM == 4 ? 0 : (wave & 1);
    fetch(0);
    stash(0, 0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < g.K; k0 += 32, buf ^= 1) {
        const bool more = k0 + 32 < g.K;
        if (more) fetch(k0 + 32);
        const float* ar = &As[buf][(32 * wt + col) * 32];
        const float* br = &Bs[buf][(32 * wn + col) * 32];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = ((2 * i + hf) ^ (col & 7)) << 2;            // (rows 32 apart: the same places)
            const float4 av = *reinterpret_cast<const float4*>(ar + at);
            float4 bv[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) bv[n] = *reinterpret_cast<const float4*>(br + 32 * 32 * n + at);
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv[n].x, acc[n], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < NT; ++n) odd[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv[n].y, odd[n], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv[n].z, acc[n], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < NT; ++n) odd[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv[n].w, odd[n], 0, 0, 0);
        }
        if (more) {
            stash(buf ^ 1, k0 + 32);              // (read last in the round before, and that round's barrier has passed)
            __syncthreads();
        }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] += odd[n][v];
    // lane = feature, register v = token 8 (v / 4) + 4 hf + v % 4 of the wavefront's 32: 128-byte runs per token.  FULL: all
    // of its tokens exist (the checks are branches around every store otherwise)
    const int tw = t0 + 32 * wt;
    if (tw >= g.tokens) return;                                  // (no barrier after this point)
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
        for (int n = 0; n < NT; ++n) {
            const int f = n0 + 32 * (wn + n) + col;
            if (f >= g.N) continue;
            if constexpr (PROJ) {
                const int seg = f / g.Hd;
                const float bias = seg == 3 ? to_f32<T>(((const T*)g.bvec)[f - 3 * g.Hd]) : 0.f;
                T* dst = (T*)g.cdst + (size_t)tw * g.N + f;
                if (seg == 3) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[n][v] = 1.f / (1.f + __expf(-(acc[n][v] + bias)));
                } else {
                    const float scale = seg == 0 ? g.qscale : 1.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[n][v] *= scale;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int x = 8 * (v >> 2) + 4 * hf + (v & 3);
                    if (FULL || tw + x < g.tokens) dst[(size_t)x * g.N] = from_f32<T>(acc[n][v]);
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

// ---------------------------------------------------------------------------------------
// Attention: a wavefront per 32 queries of one (batch row, head), up to eight of them in a block, which shares the keys
// and values of that (row, head) through LDS, `keys` of them at a time (all of them for lengths up to 256 at d = 32:
// then every load of the block is in flight together and two barriers are all it needs).  S^T = K Q^T puts a query
// in a lane: maximum and sum are lane-local but for one exchange between the halves, and register v of the
// exponentiated tile is the B operand of instruction v of O^T = V^T P^T as it stands (its two halves hold the keys
// 8 (v / 4) + v % 4 and that + 4).  The bias is added to the finished products (as the accumulator's starting value it was rounded
// with every one of them), the key mask (0 or -inf) selects.  Online softmax; a query without any unmasked key gets
// zero context.  Output o = gate * context.
struct GenericAttnArgs {
    const void* qkvg;
    const float* bias;       // [H][L][Lb] or NULL
    const float* mask;
    int64_t sr, sl;
    int r0, rows, L, Lb, H, d, keys;
    void* o;
};

template <int DG>
constexpr size_t attn_key_bytes() { return (size_t)(8 * DG + 4 + 8 * DG + 1) * 4; }      // k (padded), v, mask term

template <typename T, bool VEC, int DG>      // DG: head dimension in groups of 8 channels (rounded up)
__global__ __launch_bounds__(512) void k_attn_generic(GenericAttnArgs a) {
    constexpr int DP = 8 * DG, KP = DP + 4, NE = (DP + 31) / 32;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* s_k = smem;                               // [keys][KP]
    float* s_v = s_k + (size_t)a.keys * KP;          // [keys][DP]
    float* s_m = s_v + (size_t)a.keys * DP;          // [keys] 0 or -inf
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5, nthreads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rl = blockIdx.x / a.H, h = blockIdx.x - rl * a.H;
    const int q0 = (blockIdx.y * (nthreads >> 6) + wave) * 32, qi = q0 + col;
    const bool active = q0 < a.L;
    const int qc = qi < a.L ? qi : a.L - 1;
    const int Hd = a.H * a.d, N4 = 4 * Hd;
    const T* base = (const T*)a.qkvg + (size_t)rl * a.L * N4 + (size_t)h * a.d;

    float4 qf[DG];                                   // channels 8 i + 4 hf .. + 3 of the lane's query
#pragma unroll
    for (int i = 0; i < DG; ++i) qf[i] = load4<T, VEC>(base + (size_t)qc * N4, 8 * i + 4 * hf, a.d);
    const float* brow = a.bias ? a.bias + ((size_t)h * a.L + qc) * a.Lb : nullptr;
    const float* mask_row = a.mask ? a.mask + (int64_t)(a.r0 + rl) * a.sr : nullptr;
    f32x16 acc[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    float m = -INFINITY, sum = 0.f;

    for (int c0 = 0; c0 < a.L; c0 += a.keys) {
        const int nk = a.L - c0 < a.keys ? a.L - c0 : a.keys, nkp = (nk + 31) & ~31;
        if (c0) __syncthreads();                     // every wavefront is done with the keys before
        constexpr int PR = DP / 4;                   // pieces of a row
        for (int id = tid; id < nkp * PR; id += nthreads) {
            const int k = id / PR, e = 4 * (id - k * PR);
            float4 kv = make_float4(0.f, 0.f, 0.f, 0.f), vv = kv;
            if (k < nk) {
                const T* row = base + (size_t)(c0 + k) * N4;
                const float mk = mask_row ? mask_row[(int64_t)(c0 + k) * a.sl] : 1.f;
                kv = load4<T, VEC>(row + Hd, e, a.d);
                vv = load4<T, VEC>(row + 2 * Hd, e, a.d);
                vv = keep4(mk != 0.f, vv);           // (what a masked token holds may be anything, and 0 x NaN is NaN)
            }
            *reinterpret_cast<float4*>(s_k + k * KP + e) = kv;
            *reinterpret_cast<float4*>(s_v + k * DP + e) = vv;
        }
        for (int k = tid; k < nkp; k += nthreads) {
            bool ok = k < nk;
            if (ok && mask_row) ok = mask_row[(int64_t)(c0 + k) * a.sl] != 0.f;
            s_m[k] = ok ? 0.f : -INFINITY;
        }
        __syncthreads();
        if (!active) continue;
        for (int kt = 0; kt < nkp; kt += 32) {
            // lane = query, register 4 g + e = key kt + 8 g + 4 hf + e
            f32x16 s;
            float4 bias[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int k = kt + 8 * g + 4 * hf;
                bias[g] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (brow && c0 + k < a.Lb) bias[g] = *reinterpret_cast<const float4*>(brow + c0 + k);
                s[4 * g] = s[4 * g + 1] = s[4 * g + 2] = s[4 * g + 3] = 0.f;
            }
            const float* kr = s_k + (kt + col) * KP + 4 * hf;
#pragma unroll
            for (int i = 0; i < DG; ++i) {
                const float4 kf = *reinterpret_cast<const float4*>(kr + 8 * i);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.x, qf[i].x, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.y, qf[i].y, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.z, qf[i].z, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.w, qf[i].w, s, 0, 0, 0);
            }
            float tmax = -INFINITY;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 m4 = *reinterpret_cast<const float4*>(s_m + kt + 8 * g + 4 * hf);
                // (a select, not a sum: what the padded end of a bias row holds may be anything)
                s[4 * g] = m4.x == 0.f ? s[4 * g] + bias[g].x : m4.x;
                s[4 * g + 1] = m4.y == 0.f ? s[4 * g + 1] + bias[g].y : m4.y;
                s[4 * g + 2] = m4.z == 0.f ? s[4 * g + 2] + bias[g].z : m4.z;
                s[4 * g + 3] = m4.w == 0.f ? s[4 * g + 3] + bias[g].w : m4.w;
#pragma unroll
                for (int e = 0; e < 4; ++e) tmax = fmaxf(tmax, s[4 * g + e]);
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            const float m_new = fmaxf(m, tmax), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2f(m - ref);
            m = m_new;
            float part = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = exp2f(s[v] - ref);
                part += s[v];
            }
            sum = sum * alpha + part;
            f32x16 pv[NE];                           // the tile's own sums, so that 32 keys and the tiles round, not all keys in a row
#pragma unroll
            for (int n = 0; n < NE; ++n)
#pragma unroll
                for (int v = 0; v < 16; ++v) pv[n][v] = 0.f;
            // lane = channel 32 n + col (channels beyond DP read the row's neighbours and are dropped), half: keys + 4
            const float* vr = s_v + (kt + 4 * hf) * DP + (DP < 32 ? (col < DP ? col : 0) : col);
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int n = 0; n < NE; ++n)
                    pv[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[(8 * (v >> 2) + (v & 3)) * DP + 32 * n], s[v], pv[n], 0, 0, 0);
#pragma unroll
            for (int n = 0; n < NE; ++n)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[n][v] = fmaf(acc[n][v], alpha, pv[n][v]);
        }
    }
    if (!active || qi >= a.L) return;
    sum += __shfl_xor(sum, 32, 64);
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

// token statistics of `rows` batch rows from r0 on, and the pair bias if `pairs`
template <typename T>
static ff_status rows_t(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const Workspace& ws, int r0,
                        int rows, bool pairs, hipStream_t st) {
    RowsArgs a{};
    a.H = p.H; a.L = p.L; a.Lb = bias_pitch(p.L); a.bias = ws.bias; a.eps = p.eps;
    a.x = x; a.sr = p.sr; a.sl = p.sl; a.c = p.c; a.r0 = r0; a.tokens = rows * p.L; a.stats = ws.stats;
    bool vec = p.c % 4 == 0 && aligned_to(x, 4 * sizeof(T));
    if (pairs) {
        if (p.mode == FF_MSA_ROW) {
            a.src = z; a.sq = p.L; a.sk = 1; a.cp = p.c_z; a.g = w.lnz_g; a.b = w.lnz_b;
        } else {
            a.src = x; a.sq = p.sr; a.sk = p.sl; a.cp = p.c; a.g = w.ln_g; a.b = w.ln_b;
        }
        a.wb = w.w_b;
        a.pair_blocks = (int)(((int64_t)p.L * p.L + 31) / 32);
        vec = vec && a.cp % 4 == 0 && aligned_to(a.src, 4 * sizeof(T)) && aligned_to(a.g, 4 * sizeof(T)) && aligned_to(a.b, 4 * sizeof(T)) &&
              aligned_to(a.wb, 4 * sizeof(T));
    }
    const dim3 grid((unsigned)(a.pair_blocks + (a.tokens + 31) / 32));
    if (vec) hipLaunchKernelGGL((k_rows_generic<T, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_rows_generic<T, false>), grid, dim3(256), 0, st, a);
    return check_launch("rows (generic)");
}

template <typename T, bool PROJ>
static void launch_gemm(const GenericGemmArgs& g, bool vec, hipStream_t st) {
    const unsigned ny = (unsigned)((g.N + 63) / 64);
    // 128 tokens per block where that gives at least four blocks per compute unit, else 64.  (64 x 155 tokens, 256
    // channels: projections 59 us with 128 tokens, 64 with 64; output projection, with a quarter of the blocks, 20 us with 64)
    const bool big = (int64_t)((g.tokens + 127) / 128) * ny >= 4 * compute_units();
#define FF_GEN_GEMM(VECV)                                                                                                         \
    do {                                                                                                                          \
        if (big) hipLaunchKernelGGL((k_gemm_generic<T, PROJ, VECV, 4>), dim3((g.tokens + 127) / 128, ny), dim3(256), 0, st, g);    \
        else hipLaunchKernelGGL((k_gemm_generic<T, PROJ, VECV, 2>), dim3((g.tokens + 63) / 64, ny), dim3(256), 0, st, g);          \
    } while (0)
    if (vec) FF_GEN_GEMM(true);
    else FF_GEN_GEMM(false);
#undef FF_GEN_GEMM
}

template <typename T, bool VEC, int DG>
static ff_status launch_attn(GenericAttnArgs a, hipStream_t st) {
    // as many keys at a time as 72 KiB hold (two blocks per compute unit), a multiple of 32
    const int lp = (a.L + 31) & ~31;
    int keys = (int)(72 * 1024 / attn_key_bytes<DG>()) & ~31;
    if (keys > lp) keys = lp;
    a.keys = keys;
    const size_t smem = attn_key_bytes<DG>() * keys;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_generic<T, VEC, DG>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 72 * 1024);
    if (attr != hipSuccess) return fail(FF_EHIP, "k_attn_generic: dynamic LDS limit: %s", hipGetErrorString(attr));
    const int tiles = lp / 32;
    const int groups = (tiles + 7) / 8, waves = (tiles + groups - 1) / groups;
    hipLaunchKernelGGL((k_attn_generic<T, VEC, DG>), dim3((unsigned)(a.rows * a.H), groups), dim3(64 * waves), smem, st, a);
    return FF_OK;
}

template <typename T>
static ff_status chunk_t(const Problem& p, const ff_attn_weights& w, const void* x, const float* mask, const void* res,
                         void* out, const Workspace& ws, int r0, int rows, hipStream_t st) {
    const int tokens = rows * p.L;
    const size_t al = 4 * sizeof(T);
    GenericGemmArgs g{};
    g.a = x; g.sr = p.sr; g.sl = p.sl; g.L = p.L; g.r0 = r0; g.tokens = tokens;
    g.K = p.c; g.N = 4 * p.Hd; g.stats = ws.stats; g.ln_g = w.ln_g; g.ln_b = w.ln_b;
    g.w[0] = w.w_q; g.w[1] = w.w_k; g.w[2] = w.w_v; g.w[3] = w.w_g; g.bvec = w.b_g; g.Hd = p.Hd;
    g.qscale = kLog2e / sqrtf((float)p.d);
    g.cdst = ws.qkvg;
    launch_gemm<T, true>(g, p.c % 4 == 0 && aligned_to(x, al) && aligned_to(w.ln_g, al) && aligned_to(w.ln_b, al) && aligned_to(w.w_q, al) &&
                                aligned_to(w.w_k, al) && aligned_to(w.w_v, al) && aligned_to(w.w_g, al), st);

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
    const int rows = ws.chunk < p.R ? ws.chunk : p.R;
    return p.dtype == FF_F32 ? gen::rows_t<float>(p, w, x, z, ws, 0, rows, p.has_bias, stream)
                             : gen::rows_t<bf16_t>(p, w, x, z, ws, 0, rows, p.has_bias, stream);
}

ff_status generic_chunk(const Problem& p, const ff_attn_weights& w, const void* x, const float* mask,
                        const void* res, void* out, const Workspace& ws, int r0, int rows, hipStream_t stream) {
    if (r0 > 0) {
        const ff_status st = p.dtype == FF_F32 ? gen::rows_t<float>(p, w, x, nullptr, ws, r0, rows, false, stream)
                                               : gen::rows_t<bf16_t>(p, w, x, nullptr, ws, r0, rows, false, stream);
        if (st != FF_OK) return st;
    }
    return p.dtype == FF_F32 ? gen::chunk_t<float>(p, w, x, mask, res, out, ws, r0, rows, stream)
                             : gen::chunk_t<bf16_t>(p, w, x, mask, res, out, ws, r0, rows, stream);
}

}  // namespace ff
