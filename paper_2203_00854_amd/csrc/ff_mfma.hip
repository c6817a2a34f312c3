// bfloat16 matrix-core kernel family for gfx950 (wave64, v_mfma_f32_32x32x16_bf16).
//
// Pipeline per call (FastFold Sections 2.1, 2.3, 5.2):
//   k_prep      once per call: folds the LayerNorm gain into the merged q|k|v|gate(|bias)
//               weight matrix (Section 5.2 "merge GEMM"), with per-feature sums so that the
//               LayerNorm can be finished in the GEMM epilogue
//   k_gemm<PROJ> merged projection straight from the raw input: with W' = W*gamma,
//               LN(x) W^T = rstd * (x W'^T - mean * rowsum(W') + std * W beta), so the matrix cores
//               read x as it lies in HBM; the mean and offset terms are one extra contraction
//               step (operands split into bf16 hi + lo pairs) and the epilogue is a multiplication
//               by rstd: q scaled, gate = sigmoid(. + b_g), q,k,gate head-major, v transposed,
//               pair-bias columns as float32 [H][Lq][Lp]
//   k_attn_rows (ff_attn_rows.hip) flash-style attention: S^T = K Q^T on the matrix cores with the bias tile as
//               accumulator input, exponentials, O^T = V^T P^T; gate product
//               (the paper's fused scale + mask + bias softmax, Section 5.2, without ever
//               materialising the score tensor of Section 3.2)
//   k_gemm<OUT> output projection + b_o, scattered to the caller's layout
//   k_proj_attn sequences of 129..256 positions at head dimension 32: k_gemm<PROJ> and the attention in one
//               kernel (a block = two batch rows x one head), q, k, v and gate never leave the chip
//
// Matrix-core operand layouts (wave64, 32x32x16, bf16 in, f32 out):
//   A (32 x 16): lane l holds row l%32, columns 8*(l/32) .. +7
//   B (16 x 32): lane l holds column l%32, rows 8*(l/32) .. +7
//   C/D (32 x 32): lane l holds column l%32, register v holds row 8*(v/4) + 4*(l/32) + v%4
// Computing S^T (keys x queries) puts one query in one lane, so softmax statistics are
// lane-local except for one exchange between the two half-waves, and the exponentiated tile
// already has the B-operand layout of the second contraction once the key order inside a
// 32-key tile is permuted; the same permutation is applied when K rows and V^T columns are
// fetched, so nothing moves between the two contractions.
//
// Workspace layout of this family (Lp = Lq = L rounded up to 32, token p = rl*Lp + l):
//   bias [H][Lq][Lp] float32 (times log2 e) in 32 x 32 tiles (bias_index); rows of pad queries are never written nor read: their
//   lanes take the last real query's (a NaN there would reach the denominators of others, see add_piece)
//   q, k, g, o [rows][H][Lp][D] bf16;  vt [rows][H][Lp/32][D][32] bf16
//   prepared weights [(4*Hd + 32)][c] (+ [32][c_z] in row mode) bf16, their sums and offsets
// Pad tokens (l in [L, Lp)) hold finite values everywhere; they are masked as keys.
#include "ff_attn_rows.h"
#include "ff_common.h"

#include <math.h>

#include <type_traits>

namespace ff {

__device__ __forceinline__ float bf16_round(float f) { return lo_f32(pack2(f, 0.f)); }

__device__ __forceinline__ uint4 ldg16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ uint2 ldg8(const void* p) { return *reinterpret_cast<const uint2*>(p); }
// (see ldg16 with a base and an offset per lane)
__device__ __forceinline__ uint2 ldg8(const void* base, uint32_t lane_bytes) {
    return *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(base) + lane_bytes);
}
__device__ __forceinline__ void stg16(void* base, uint32_t lane_bytes, uint4 v) {
    *reinterpret_cast<uint4*>(reinterpret_cast<char*>(base) + lane_bytes) = v;
}

// sum of the squares of the two bf16 halves of w, added to acc (v_dot2c_f32_bf16: exact products)
__device__ __forceinline__ float add_pair_sq(uint32_t w, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, w), acc, false);
}

// LayerNorm statistics of a token whose K channels lie in the KC fragments of the two lanes
// (col, hf = 0 | 1), channels beyond K being zero: mean and variance + eps, float32, in one pass
// over the registers.  sum x and sum x^2 are accumulated from exact bf16 products (two channels
// per instruction), var = sum x^2 / K - mean^2: the cancellation costs a relative error of
// about 2^-22 (1 + mean^2 / var) of the variance, 2e-5 for a mean of twelve standard
// deviations.  (The two-pass form, sum (x - mean)^2, took 450 vector instructions per lane for
// K = 256, a quarter of this wavefront's work before its first matrix instruction.)
// Every kernel takes the statistics from here, so that they agree bit for bit.
template <int KC>
__device__ __forceinline__ void token_stats(const Frag (&xa)[KC], int K, float eps, float& mu, float& var) {
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int s = 0; s < KC; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sum = add_pair(xa[s].w[i], sum);
            sq = add_pair_sq(xa[s].w[i], sq);
        }
    sum += other_half(sum);
    sq += other_half(sq);
    const float inv_k = 1.f / (float)K;
    mu = sum * inv_k;
    var = fmaxf(sq * inv_k - mu * mu, 0.f) + eps;
}

static inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

// ------------------------------------------------------------------------------------
struct MfmaWs {
    bf16_t *q, *k, *g, *vt, *o;
    bf16_t *wp, *zwp;      // prepared weights: main [(4Hd+32)][c], row-mode bias [32][c_z]
    uint4* aug;            // [(4Hd+32) + 32] per row of wp / zwp: its sum and output offset as bf16 pairs (see k_prep)
};

static MfmaWs split_ws(const Problem& p, int chunk, const Workspace& ws) {
    const size_t Lp = round_up(p.L, 32);
    const size_t n = (size_t)chunk * Lp * p.Hd;   // elements per tensor
    MfmaWs m;
    m.q = (bf16_t*)ws.qkvg;
    m.k = m.q + n;
    // The gate between k and v^T, not behind them in the order of the feature tiles: k_attn_rows streams k and v^T at the same time, and with
    // the two next to each other it draws more power for the same cycles and bytes, so a card at its power limit runs it at a lower
    // clock (1024 x 384 tokens, 64 channels, head dim 8, called over and over on such a card: 436 us next to each other, 431 apart).
    m.g = m.k + n;
    m.vt = m.g + n;
    m.o = (bf16_t*)ws.o;
    char* pr = (char*)ws.prep;
    const size_t rows_main = 4 * (size_t)p.Hd + 32;
    m.wp = (bf16_t*)pr;
    pr += align256(rows_main * p.c * 2);
    m.zwp = (bf16_t*)pr;
    pr += align256((size_t)32 * (p.c_z > 0 ? p.c_z : 1) * 2);
    m.aug = (uint4*)pr;
    return m;
}

bool mfma_supported(const Problem& p) {
    if (p.dtype != FF_BF16) return false;
    if (p.c % 32 != 0 || p.c > 256) return false;
    if (p.Hd % 32 != 0 || p.Hd > 256) return false;
    if (p.d != 8 && p.d != 16 && p.d != 32) return false;
    if (p.L > 16384) return false;
    if (p.H > 32) return false;
    if (p.mode == FF_MSA_ROW && (p.c_z % 16 != 0 || p.c_z > 256)) return false;
    return true;
}

size_t mfma_workspace(const Problem& p, int chunk, Workspace* ws, void* base) {
    const size_t Lp = round_up(p.L, 32), Lq = round_up(p.L, 32);
    size_t off = 0;
    char* b = (char*)base;
    ws->bias = nullptr;
    if (p.has_bias) {
        ws->bias = (float*)(b + off);
        off += align256((size_t)p.H * Lq * Lp * 4);
    }
    const size_t n = (size_t)chunk * Lp * p.Hd * 2;
    ws->stats = nullptr;
    ws->qkvg = b + off;
    off += align256(4 * n);
    ws->o = b + off;
    off += align256(n);
    ws->prep = b + off;
    const size_t rows_main = 4 * (size_t)p.Hd + 32;
    off += align256(rows_main * p.c * 2) + align256((size_t)32 * (p.c_z > 0 ? p.c_z : 1) * 2) +
           align256((rows_main + 32) * 16);
    ws->total = off;
    ws->chunk = chunk;
    return off;
}

// ====================================================================================
// Weight preparation: one wavefront per output row n of the merged matrix.
//   wp[n][k] = bf16(scale * W[n][k] * gamma[k]);  sn[n] = sum_k wp[n][k];
//   cn[n] = scale * sum_k W[n][k] * beta[k] (+ extra[n])
// sn and cn leave as one extra 8-slot piece of the contraction per row, split into bf16 pairs
// (hi + lo): [sn_hi, sn_lo, sn_hi, cn_hi, cn_lo, cn_hi, 0, 0].  Against the token's piece
// [m_hi, m_hi, m_lo, r_hi, r_hi, r_lo, 0, 0] (m = -mean, r = standard deviation) the matrix core
// adds -mean*sn + r*cn to x W'^T, so that the GEMM epilogue is one multiplication by 1/r.
struct PrepSeg {
    const bf16_t* w;              // [rows][K]
    const bf16_t* extra;          // [rows] added to cn, or NULL
    const bf16_t *gamma, *beta;   // [K]
    bf16_t* wp;                   // output rows of this segment [rows_pad][K]
    uint4* aug;                   // [rows_pad]
    int rows, rows_pad, K;        // rows_pad - rows zero rows follow
    float scale;
};
struct PrepArgs {
    PrepSeg seg[6];
    int nseg;
};

// One row of a folded matrix by one wavefront: store(k, bf16(scale * w[k] * gamma[k])) for k < K and
// the row's extra piece as the return value (valid in every lane).  Every kernel that folds a row
// goes through here, so that the same weights give the same bits wherever they are prepared (the
// pair bias of the triangle modes is prepared by k_prep when it rides along with the projections
// and by k_prep_bias when the rows are chunked, and both must give the same output bits).
struct FoldRow {
    bf16_t w[4], g[4], b[4];
};
__device__ __forceinline__ FoldRow fold_load(const bf16_t* wrow, const bf16_t* gamma, const bf16_t* beta, int K, int lane) {
    FoldRow f;
    // K <= 256: at most four elements per lane.  The loads carry no condition (an element beyond K
    // reads element K - 1 and is dropped below, a pad row reads the row the caller passes for it): a
    // conditional load is a branch and a wait of its own, twelve memory round trips one after the other
    // instead of one.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = lane + 64 * i;
        const int kc = k < K ? k : K - 1;
        f.w[i] = wrow[kc];
        f.g[i] = gamma[kc];
        f.b[i] = beta[kc];
    }
    return f;
}
template <typename Store>
__device__ __forceinline__ uint4 fold_row(FoldRow f, int K, float scale, bool real, float extra, int lane, Store&& store) {
    float sum = 0.f, cst = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool in = real && lane + 64 * i < K;
        if (!in) f.w[i] = f.g[i] = f.b[i] = (bf16_t)0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = lane + 64 * i;
        if (k < K) {
            const float w = bf16_to_f32(f.w[i]) * scale;
            const float r = bf16_round(w * bf16_to_f32(f.g[i]));
            cst += w * bf16_to_f32(f.b[i]);
            store(k, f32_to_bf16(r));
            sum += r;
        }
    }
    sum = wave_sum(sum);
    cst = wave_sum(cst);
    const float cn = cst + extra;
    const float sn_hi = bf16_round(sum), sn_lo = bf16_round(sum - sn_hi);
    const float cn_hi = bf16_round(cn), cn_lo = bf16_round(cn - cn_hi);
    return make_uint4(pack2(sn_hi, sn_lo), pack2(sn_hi, cn_hi), pack2(cn_lo, cn_hi), 0u);
}

// row n of the concatenated segments, by one wavefront
__device__ __forceinline__ void prep_row(const PrepArgs& a, int n_in, int lane) {
    const int n = __builtin_amdgcn_readfirstlane(n_in);      // (a wavefront's row: the segment is then read with scalar loads)
    int base = 0, sg = -1, local = 0;
    for (int i = 0; i < a.nseg; ++i) {
        if (sg < 0 && n < base + a.seg[i].rows_pad) {
            sg = i;
            local = n - base;
        }
        base += a.seg[i].rows_pad;
    }
    if (sg < 0) return;
    PrepSeg sgm = a.seg[0];
#pragma unroll
    for (int i = 1; i < 6; ++i)
        if (i == sg) sgm = a.seg[i];
    const bool real = local < sgm.rows;
    const int K = sgm.K;
    // (no condition on the load, see fold_load: without an offset vector the row reads gamma[0] and drops it)
    const bool has_extra = real && sgm.extra != nullptr;
    const float extra_raw = bf16_to_f32(*(has_extra ? sgm.extra + local : sgm.gamma));
    const float extra = has_extra ? extra_raw : 0.f;
    bf16_t* wp = sgm.wp + (size_t)local * K;
    // (a pad row has no weights, its segment possibly no matrix at all: it reads gamma, K valid elements, instead)
    const uint4 piece = fold_row(fold_load(real ? sgm.w + (size_t)local * K : sgm.gamma, sgm.gamma, sgm.beta, K, lane), K, sgm.scale, real, extra, lane,
                                 [&](int k, bf16_t v) { wp[k] = v; });
    if (lane == 0) sgm.aug[local] = piece;
}

__global__ __launch_bounds__(256) void k_prep(PrepArgs a) {
    prep_row(a, blockIdx.x * 4 + (threadIdx.x >> 6), threadIdx.x & 63);
}

// ====================================================================================
// The pair bias b[h][i][j] = log2(e) * sum_c LN(z[i][j])_c W_b[h][c] as a pass of its own (row mode:
// over the pair representation with its own LayerNorm; chunked triangle modes: over all of x before
// the first chunk) and the weight preparation in ONE launch (they do not depend on each other).  Blocks below bias_blocks take
// 256 pairs each (one 32-pair tile per wavefront, the folded 32 x K weight tile built by the block
// itself in LDS, same algebra as k_gemm's pair-bias tile); the blocks above them run prep_row.
// Element (h, q, k) of the pair bias [H][Lq][Lp]: 32 x 32 tiles in the register order of an S^T accumulator,
// [H][Lq/32][Lp/32][4][64 lanes][4]: lane = (q % 32) + 32 hf
// holds the keys 16c + 8hf + 4i + e of the tile in element e of group 2c + i, so that a wavefront
// fetches a tile with four loads of 1 KiB each.
__device__ __forceinline__ size_t bias_index(int h, int q, int k, int Lq, int Lp) {
    const int kk = k & 31;
    const int grp = 2 * (kk >> 4) + ((kk >> 2) & 1), hf = (kk >> 3) & 1;
    const size_t tile = ((size_t)h * (Lq >> 5) + (q >> 5)) * (Lp >> 5) + (k >> 5);
    return ((tile * 4 + grp) * 64 + (q & 31) + 32 * hf) * 4 + (kk & 3);
}

struct PrepBiasArgs {
    PrepArgs prep;
    int bias_blocks;
    const bf16_t* z;             // pair (i, j) at z + (i*sr + j*sl)*K
    int64_t sr, sl;
    const bf16_t *w_b, *gamma, *beta;   // [H][K], [K], [K]
    float* bias;                 // [H][Lq][Lp]
    int L, Lp, Lq, K, H;
    float eps;
};

template <int KC>
__global__ __launch_bounds__(512) void k_prep_bias(PrepBiasArgs a) {
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= a.bias_blocks) {
        prep_row(a.prep, ((int)blockIdx.x - a.bias_blocks) * 8 + wave, lane);
        return;
    }
    constexpr int PITCH = KC * 32 + 16;                 // bytes per weight row in LDS (padded: conflict-free reads)
    __shared__ __attribute__((aligned(16))) unsigned char s_w[32 * PITCH];
    __shared__ uint4 s_aug[32];
    const int K = a.K;

    // ---- the weights of this wavefront's first head row, requested ahead of the pairs (a wait for them, had they been requested
    // later, would be one for the pairs as well): the row is folded while the pairs are under way.  With it and without conditions on the pairs'
    // loads 8 x 700 row attention of 16 heads 76.7 -> 74.5 us, 60 x 300 59.9 -> 59.1, 128 x 256 61.0 -> 59.9; chunked triangle attention at 2048 the same.
    const FoldRow first = fold_load(a.w_b + (size_t)(wave < a.H ? wave : 0) * K, a.gamma, a.beta, K, lane);
    __builtin_amdgcn_sched_barrier(0);

    // ---- pairs of this wavefront: raw operand fragments
    const int tiles_m = a.L * (a.Lp >> 5);
    int tg = blockIdx.x * 8 + wave;
    if (tg > tiles_m - 1) tg = tiles_m - 1;             // (repeats the last tile: same values stored twice)
    const int pr = tg * 32 + col;
    const int qi = pr / a.Lp, kj = pr - qi * a.Lp;
    const bool valid = kj < a.L;
    // Eight lanes fetch one 128-byte line of a pair (64 channels); the lines pass through 4 KiB of LDS
    // per wavefront and come back in the operand layout (lane = pair, pieces 2s' + hf of line m =
    // contraction steps 4m + s').  A load with lane = pair touches 64 cache lines for 1 KiB, and the
    // cache looks up one line per cycle: the fetch alone took 2.5 us of the block's 6.
    constexpr int NG = (KC + 3) / 4;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[8][4096];
    unsigned char* s_st = s_stage[wave];
    // The loads carry no condition (pieces outside repeat one that exists and are cleared at their arrival): each would wait for itself.
    uint4 raw[NG][4];
    const int pieces = K >> 3;
    const int q0 = (tg * 32) / a.Lp, k0 = tg * 32 - q0 * a.Lp;           // (uniform: a tile lies inside one query row)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int kk = k0 + 8 * i + (lane >> 3);
        const bf16_t* zq = a.z + ((int64_t)q0 * a.sr + (int64_t)(kk < a.L ? kk : 0) * a.sl) * K;
#pragma unroll
        for (int m = 0; m < NG; ++m) {
            const int pc = 8 * m + (lane & 7);
            raw[m][i] = ldg16(zq + 8 * (pc < pieces ? pc : 0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- the folded weight tile: zeros, then one wavefront per head row (fold_row)
    for (int i = tid; i < 32 * PITCH / 16; i += 512) reinterpret_cast<uint4*>(s_w)[i] = make_uint4(0, 0, 0, 0);
    if (tid < 32) s_aug[tid] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (int row = wave; row < a.H; row += 8) {
        bf16_t* dst = reinterpret_cast<bf16_t*>(&s_w[row * PITCH]);
        const uint4 piece = fold_row(row == wave ? first : fold_load(a.w_b + (size_t)row * K, a.gamma, a.beta, K, lane), K, kLog2e, true, 0.f, lane,
                                     [&](int k, bf16_t v) { dst[k] = v; });
        if (lane == 0) s_aug[row] = piece;
    }

    if (k0 + 32 > a.L || NG * 8 != pieces) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = k0 + 8 * i + (lane >> 3) < a.L;
#pragma unroll
            for (int m = 0; m < NG; ++m)
                if (!in || 8 * m + (lane & 7) >= pieces) raw[m][i] = make_uint4(0, 0, 0, 0);
        }
    }
    // ---- the pairs as operands (the staging area is the wavefront's own, its LDS operations complete in order)
    Frag xa[KC];
#pragma unroll
    for (int m = 0; m < NG; ++m) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tl = 8 * i + (lane >> 3);
            *reinterpret_cast<uint4*>(s_st + tl * 128 + (((lane & 7) ^ (tl & 7)) * 16)) = raw[m][i];
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
            if (4 * m + sp < KC)
                xa[4 * m + sp].u = *reinterpret_cast<const uint4*>(s_st + col * 128 + (((2 * sp + hf) ^ (col & 7)) * 16));
        __builtin_amdgcn_wave_barrier();
    }

    // ---- LayerNorm statistics of the wavefront's pairs
    float mu, var;
    token_stats<KC>(xa, K, a.eps, mu, var);
    const float rstd = valid ? rsqrtf(var) : 0.f;
    const float m = valid ? -mu : 0.f, r = var * rstd;
    const float m_hi = bf16_round(m), m_lo = bf16_round(m - m_hi);
    const float r_hi = bf16_round(r), r_lo = bf16_round(r - r_hi);
    Frag xaug;
    xaug.u = make_uint4(0, 0, 0, 0);
    if (hf == 0) xaug.u = make_uint4(pack2(m_hi, m_hi), pack2(m_lo, r_hi), pack2(r_hi, r_lo), 0u);

    __syncthreads();
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int s = 0; s < KC; ++s) {
        Frag wf;
        wf.u = *reinterpret_cast<const uint4*>(&s_w[col * PITCH + (2 * s + hf) * 16]);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf.v, xa[s].v, acc, 0, 0, 0);
    }
    {
        Frag wa;
        wa.u = s_aug[col];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa.v, xaug.v, acc, 0, 0, 0);
    }
    // lane = pair (qi, kj), register v = head 8*(v/4) + 4*hf + v%4
    float* bp = a.bias + bias_index(0, qi, kj, a.Lq, a.Lp);
    const size_t plane = (size_t)a.Lq * a.Lp;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int h = 8 * (v >> 2) + 4 * hf + (v & 3);
        if (h < a.H) bp[(size_t)h * plane] = acc[v] * rstd;
    }
}

// ====================================================================================
// GEMM with the whole contraction length (<= 256) resident: a wavefront owns a 32-token tile as register-resident operand fragments
// and sweeps over 32-feature tiles of the weight matrix, which the block keeps in LDS: all of them where they fit (no barrier after the
// first, the wavefronts of the grid walk over the token tiles by themselves), else two halves of NS tiles each, one being
// worked on while the other is filled (global_load_lds_dwordx4: lane i of a wavefront deposits its 16 bytes at the
// wave-uniform LDS base + 16 i).
// What bounds it is the number of instructions a wavefront can issue (one every eight cycles or so, whatever the others do): a q or k tile at 128
// channels passes 170, 9 of them matrix instructions, 82 vector, LDS and memory instructions, the rest scalar ones, waits and branches.  So the
// registers are held to 128, sixteen wavefronts per compute unit, and a wavefront finishes a
// tile before it begins the next one: the matrix instructions of one hide behind the epilogues of the other three of its SIMD.  (A kernel of
// eight wavefronts with 186 to 250 registers that alternated the matrix instructions of a tile with the epilogue of the one before: whole calls of
// triangle attention at 333 117 us, now 104; 60 x 300 row attention 75, now 60; 300 x 48 columns 52, now 46.)  The projections of 64 x 2048
// tokens of 128 channels take 34 to 36 us, 0.21 of the matrix rate, with 88 vector and 69 scalar instructions per tile (counters).
// No instance may spill: a kernel that uses scratch memory starts 2.5 us later (8 x 48 row attention, projections 11.7 -> 9.2 us).
//
// LDS image of a tile: 32 rows of P = 2 KC 16-byte pieces, piece p of row r at slot
// r P + (p ^ g(r)); g spreads 16 consecutive rows over the 16 slots of a 256-byte LDS line, so
// the operand reads (lane = row, all lanes the same piece) are conflict free without padding.
struct GemmArgs {
    int along, split;        // blocks along the tokens, shares of the feature tiles
    uint32_t split_inv;      // 2^32 / split rounded up (split > 1): item / split as a product
    int per_xcd;             // blocks of an XCD
    int waves;               // wavefronts of a block: eight, or gemm_waves(KC)
    int ft_count;            // feature tiles of this launch
    int tiles_per_split;     // feature tiles of a share
    const bf16_t* src;     // PROJ: x or z (strided tokens); OUT: o [rows][H][Lp][D]
    int64_t sr, sl;        // token strides of src (PROJ) / out (OUT)
    int r0, rows, L, Lp, Lq;
    int K;                 // contraction length
    float eps;
    const bf16_t* w;       // PROJ: prepared weights [tiles*32][K]; OUT: w_o [N][K]
    const uint4* aug;      // PROJ: per-feature extra piece of the contraction (sum and offset, see k_prep)
    const bf16_t* bvec;    // OUT: b_o [N]
    int Hd, H, D;
    int dsh;               // log2(D), D in {8, 16, 32}
    int odd_step, even_step; // OUT: elements from an even contraction step of 16 channels to the odd one behind it, and from that to the next even one
    int nt_main;           // PROJ: 32-feature tiles of q|k|v|gate; tile nt_main is the pair-bias tile
    bf16_t* q;               // PROJ outputs: q, then k, gate and v^T, each `tensor` elements behind the one before
    int64_t tensor;
    float* bias;             // PROJ pair-bias output, [H][Lq][Lp] elements in the tiles of bias_index
    bf16_t* out;             // OUT output, token (r,l) at (r*sr + l*sl)*N
    const bf16_t* res;       // OUT with RES: added to the output, laid out like out (may be out itself)
    int N;                   // OUT: features
};

typedef void __attribute__((address_space(3)))* lptr_t;

// Wait until at most n (rounded down to 8, 4, 2 or 0) vector-memory operations of this wavefront
// are outstanding, and none of its LDS reads.  They complete in order, so with n = number of stores issued after a load this
// waits for the load but not for those stores.
__device__ __forceinline__ void wait_vmem_but_last(int n) {
    if (n >= 8) __builtin_amdgcn_s_waitcnt(0x0078);
    else if (n >= 4) __builtin_amdgcn_s_waitcnt(0x0074);
    else if (n >= 2) __builtin_amdgcn_s_waitcnt(0x0072);
    else __builtin_amdgcn_s_waitcnt(0x0070);
}

constexpr int gemm_waves(int kc) { return kc >= 16 ? 12 : 16; }    // wavefronts per compute unit: four per SIMD, three where the tokens take 64 registers
constexpr int gemm_fit(int kc, bool proj) { return proj ? gemm_waves(kc) : 16; }   // and of several blocks: the output projections keep to 128 registers at 256 channels too
constexpr int gemm_half(int kc) { return kc >= 16 ? 4 : 9; }       // NS: weight tiles per half of the ring

// dynamic LDS of k_gemm: weight tiles, 1/std of the wavefronts' tokens, per-feature offsets and extra pieces
static size_t gemm_smem_bytes(int kc, int tiles) {
    const int held = tiles < 2 * gemm_half(kc) ? tiles : 2 * gemm_half(kc);
    return (size_t)held * kc * 1024 + (size_t)gemm_waves(kc) * 32 * 4 + (size_t)tiles * 32 * (4 + 16);
}

// tile kinds of k_gemm (q and k share their epilogue)
enum { TK_Q = 0, TK_K = 1, TK_V = 2, TK_GATE = 3, TK_BIAS = 4, TK_OUT = 5 };

template <int KC, bool PROJ, bool RES>
__global__ __launch_bounds__(gemm_waves(KC) * 64, gemm_fit(KC, PROJ) / 4) void k_gemm(GemmArgs a) {
    static_assert(!(PROJ && RES), "the residual belongs to the output projection");
    constexpr int NS = gemm_half(KC);
    constexpr int P = 2 * KC;                           // 16-byte pieces per weight row
    constexpr int STAGE = 32 * P * 16;                  // bytes of one 32-feature tile in LDS
    constexpr int RSH = P >= 16 ? 0 : (P == 8 ? 1 : 2);
    constexpr int GM = (P >= 16 ? 16 : P) - 1;          // g(r) = (r >> RSH) & GM
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // Work-groups go to the 8 XCDs round-robin and each XCD has its own L2: an XCD takes a contiguous range of the order (token block,
    // share), so that the shares of the same tokens run on one XCD at the same time and every XCD has its eighth of the blocks.  (With
    // the blocks along the tokens rounded up to a multiple of 8 instead, 8 x 48 tokens were two of eight: everything ran on two XCDs
    // behind three empty blocks for each that had work.)  Projections without shares have no tokens to share and take the blocks as they
    // come, so that what the chip writes at one time lies together: eight ranges far apart leave k_attn_rows, which reads them next, 3 % slower at
    // 700 x 250 tokens of 64 channels (the call 164.0 -> 157.7 us on a card with power to spare, 172 -> 161 at its limit; 1024 x 384 405 -> 409
    // and 436 -> 423 with the order of the tensors above; within 1 % elsewhere).  The output projection keeps the ranges: so do the kernels that write its tokens.
    // (all arguments are on their way before the first one is waited for: a small call waits for little else than its chain of loads)
    asm volatile("" : : "s"(a.src), "s"(a.sr), "s"(a.sl), "s"(a.r0), "s"(a.rows), "s"(a.L), "s"(a.Lp), "s"(a.K), "s"(a.w), "s"(a.aug), "s"(a.bvec),
                 "s"(a.Hd), "s"(a.H), "s"(a.D), "s"(a.dsh), "s"(a.odd_step), "s"(a.even_step));
    const int item = (int)(blockIdx.x & 7) * a.per_xcd + (int)(blockIdx.x >> 3);
    const int block = a.split > 1 ? (int)__umulhi((unsigned)item, a.split_inv) : (PROJ ? (int)blockIdx.x : item), share = a.split > 1 ? item - block * a.split : 0;
    const int ft_begin = share * a.tiles_per_split;
    const int ft_end = ft_begin + a.tiles_per_split < a.ft_count ? ft_begin + a.tiles_per_split : a.ft_count;
    const int n_ft = ft_end - ft_begin;
    const int NW = a.waves;
    const int tiles_m = a.rows * (a.Lp >> 5);
    if (block >= a.along) return;                       // (whole block)
    const bool whole = n_ft <= 2 * NS;                                    // all of the block's weights are in LDS at once
    unsigned char* s_w = smem;                                            // [min(n_ft, 2 NS)][STAGE]
    uint4* s_aug = reinterpret_cast<uint4*>(smem + (whole ? n_ft : 2 * NS) * STAGE);      // PROJ: [n_ft][32] extra piece per feature
    float* s_cn = reinterpret_cast<float*>(s_aug + n_ft * 32);            // OUT: [n_ft][32] output bias
    float* s_rstd = s_cn + n_ft * 32;                                     // [wave][32]: 1/std of the wavefront's tokens

    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = a.K;

    // ---- token operand fragments, raw (issued first: they come from HBM)
    Frag xa[KC];
    int rl = 0, l = 0;                    // batch row (wave-uniform) and position of this lane's token
    bool valid = false;
    uint32_t ahead[2] = {0u, 0u};
    const int LpD = a.Lp * a.D;           // every tensor of this family has Lp*Hd elements per batch row
    auto load_tokens = [&](int unit) __attribute__((always_inline)) {
        const int tg = unit < tiles_m ? unit : tiles_m - 1;
        // (a tile lies inside one batch row; neighbouring wavefronts take tokens that are neighbours in memory)
        const unsigned by = (unsigned)(a.sl > a.sr ? a.rows : a.Lp >> 5);
        const int major = (int)((unsigned)tg / by), minor = tg - major * (int)by;
        rl = a.sl > a.sr ? minor : major;
        l = 32 * (a.sl > a.sr ? major : minor) + col;
        valid = l < a.L;
        // (pad tokens load the last one again: clear_pad drops it)
        const int lc = valid ? l : a.L - 1;
        // (K is a multiple of 16, so a contraction step has both of its pieces or none: what depends on the step is uniform.  Worked out step by
        // step, from an opaque K: the offsets of all steps at once do not fit the scalar registers)
        int k = K;
        asm volatile("" : "+s"(k));
        if constexpr (PROJ) {
            const bf16_t* sp = a.src + ((int64_t)(a.r0 + rl) * a.sr + (int64_t)lc * a.sl) * K + 8 * hf;
            if (k == 16 * KC) {
#pragma unroll
                for (int s = 0; s < KC; ++s) xa[s].u = ldg16(sp + 16 * s);
            } else {
#pragma unroll
                for (int s = 0; s < KC; ++s) {
                    if (16 * s < k) xa[s].u = ldg16(sp + 16 * s);
                    else xa[s].u = make_uint4(0, 0, 0, 0);
                }
            }
        } else {                                                          // gated context, head-major [row][head][l][d]
            const bf16_t* ctx = a.src + (size_t)rl * a.H * LpD;
            const uint32_t lane_at = (uint32_t)(lc * a.D + (a.D == 8 ? hf * LpD : 8 * hf)) * 2;
            if (k == 16 * KC) {
#pragma unroll
                for (int s = 0; s < KC; ++s) {
                    xa[s].u = ldg16(ctx, lane_at);
                    ctx += s & 1 ? a.even_step : a.odd_step;
                }
            } else {
#pragma unroll
                for (int s = 0; s < KC; ++s) {
                    if (16 * s < k) xa[s].u = ldg16(ctx, lane_at);
                    else xa[s].u = make_uint4(0, 0, 0, 0);
                    ctx += s & 1 ? a.even_step : a.odd_step;
                }
            }
        }
        if constexpr (RES) {
            // the residual's lines of the share into L2, a load per line (N <= 256: at most four per token): the
            // loads below come one feature tile ahead of their use, too late for memory
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int line = (lane >> 5) + 2 * i, at = ft_begin * 32 + 64 * line < ft_end * 32 ? ft_begin * 32 + 64 * line : ft_begin * 32;
                ahead[i] = *reinterpret_cast<const uint32_t*>(a.res + (size_t)(((int64_t)(a.r0 + rl) * a.sr + (int64_t)lc * a.sl) * a.N) + at);
            }
        }
    };
    // (where the tokens are waited for anyway: between their loads and those of the weights it would put one memory latency behind the other)
    auto clear_pad = [&]() __attribute__((always_inline)) {
        if (l - col + 32 > a.L) {                                        // (wave-uniform)
            const uint32_t m = valid ? 0xffffffffu : 0u;
#pragma unroll
            for (int s = 0; s < KC; ++s) xa[s].u = make_uint4(xa[s].u.x & m, xa[s].u.y & m, xa[s].u.z & m, xa[s].u.w & m);
        }
    };
    int unit = block * NW + wave;
    load_tokens(unit);

    // ---- weight tiles: KC chunks of 64 pieces (1 KiB) each, shared out over the wavefronts: chunk c of a half goes to
    // wavefront c % NW.  Pieces beyond K re-read the last valid piece (the token operand is zero there).
    const unsigned s_w_lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)s_w);
    auto issue = [&](int first, int count, int slot) __attribute__((always_inline)) {      // tiles first .. + count - 1 into the slots slot ..
        for (int c = wave; c < count * KC; c += NW) {
            const int ft = c / KC, ps = (c - ft * KC) * 64 + lane, row = ps / P;
            int kk = ((ps % P) ^ ((row >> RSH) & GM)) * 8;
            if (kk > K - 8) kk = K - 8;
            ff::load16_to_lds(a.w + (size_t)(ft_begin + first + ft) * 32 * K, (uint32_t)(row * K + kk) * 2,
                              s_w_lds + (unsigned)((slot + ft) * STAGE + (c - ft * KC) * 1024));
        }
    };
    issue(0, n_ft < 2 * NS ? n_ft : 2 * NS, 0);
    // per-feature offsets of this block's tiles
    for (int i = tid; i < n_ft * 32; i += NW * 64) {
        if constexpr (PROJ) s_aug[i] = a.aug[ft_begin * 32 + i];
        else s_cn[i] = bf16_to_f32(a.bvec[ft_begin * 32 + i]);
    }
    // operand read: piece 2s + hf of row col sits at byte rd0 ^ (32 s) of its tile
    const unsigned rd0 = (unsigned)col * (P * 16) + 16u * (unsigned)((((col >> RSH) & GM)) ^ hf);
    // lane's part of the places of a tile's two stores (see there): token or feature lane % 16 of the first or second sixteen, piece
    const int t16 = lane & 15, piece8 = 8 * (2 * ((lane >> 4) & 1) + hf);
    const unsigned t_lane = a.D == 32 ? (unsigned)t16 * 32 + piece8 : (unsigned)col * a.D + (a.D == 16 ? 8 * hf : hf * LpD);
    const unsigned t_second = a.D == 32 ? 16 * 32 : (unsigned)(16 >> a.dsh) * LpD;
    const unsigned v_lane = (unsigned)(t16 >> a.dsh) * LpD + (unsigned)(t16 & (a.D - 1)) * 32 + piece8;
    const unsigned v_second = (unsigned)((16 >> a.dsh) * LpD + (16 & (a.D - 1)) * 32);
    const int64_t o_lane = (int64_t)t16 * a.sl * a.N + piece8;

    // the share's first tile (see the loop): its kind, the tiles left of that kind, its place in the outputs of a batch row
    const int per_kind = a.nt_main >> 2, tile_step = (32 >> a.dsh) * LpD;
    const int kind0 = PROJ ? (ft_begin >= per_kind) + (ft_begin >= 2 * per_kind) + (ft_begin >= 3 * per_kind) + (ft_begin >= a.nt_main) : (int)TK_OUT;
    const int kind_left0 = (kind0 + 1) * per_kind - ft_begin;
    const int64_t to0 = (kind0 ^ (kind0 >> 1)) * a.tensor + (per_kind - kind_left0) * tile_step;

    // ---- residual (RES): the matrix core adds it.  Two more contraction steps multiply a
    // selection matrix (feature f of the tile picks slot f, then f - 16) with the residual
    // values of 16 features per token: 1.0 * bf16 into the float32 accumulator is exact, the
    // operand is the token's row as it lies in memory (16 bytes per lane, the very bytes the
    // lane stores later, so the output may replace the residual in place), and the sum is
    // rounded to bf16 once.
    Frag sel[2], rn[2];
    if constexpr (RES) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int k = col - 16 * m - 8 * hf;             // slot of this lane's feature inside its piece
#pragma unroll
            for (int i = 0; i < 4; ++i)
                sel[m].w[i] = (k >> 1) == i ? ((k & 1) ? 0x3f800000u : 0x00003f80u) : 0u;
        }
    }

    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();

    for (;; load_tokens(unit)) {
        clear_pad();
        if constexpr (RES) asm volatile("" : : "v"(ahead[0]), "v"(ahead[1]));      // (they set out with the tokens)
        const bool run = unit < tiles_m;                      // (wave-uniform; without whole weights a wavefront without tokens still takes its share of the loads)
        float rstd = 0.f;         // 1 / standard deviation of this lane's token
        Frag xaug;                // its extra piece of the contraction: (-mean, standard deviation) as bf16 pairs (see k_prep)
        xaug.u = make_uint4(0, 0, 0, 0);
        if constexpr (PROJ) {
            // LayerNorm statistics of the raw rows (token_stats)
            float mu, var;
            token_stats<KC>(xa, K, a.eps, mu, var);
            rstd = valid ? rsqrtf(var) : 0.f;
            const float m = valid ? -mu : 0.f, r = var * rstd;
            const float m_hi = bf16_round(m), m_lo = bf16_round(m - m_hi);
            const float r_hi = bf16_round(r), r_lo = bf16_round(r - r_hi);
            if (hf == 0) {
                xaug.u = make_uint4(pack2(m_hi, m_hi), pack2(m_lo, r_hi), pack2(r_hi, r_lo), 0u);
                s_rstd[wave * 32 + col] = rstd;
            }
        }
        // q, k, gate, v^T of the token tile's batch row; RES: the lane's token in out (pad tokens: the last real one, they load the residual and
        // never store)
        const size_t row_base = PROJ ? (size_t)rl * a.H * LpD
                                     : (size_t)(((int64_t)(a.r0 + rl) * a.sr + (int64_t)(valid ? l : a.L - 1) * a.sl) * a.N);
        const int l0 = __builtin_amdgcn_readfirstlane(l - col);
        auto load_res = [&](int ft) __attribute__((always_inline)) {
            if (ft > ft_end - 1) ft = ft_end - 1;            // (past the end: a harmless repeat)
            const bf16_t* rp = a.res + row_base + (size_t)ft * 32 + 8 * hf;
            rn[0].u = ldg16(rp);
            rn[1].u = ldg16(rp + 16);
        };
        if constexpr (RES) load_res(ft_begin);
        int n_ops = 0;            // stores and residual loads issued since the last weight loads (a lower bound)
        // What a tile needs of its place moves on by additions: its slot in LDS, the tiles left of its half of the ring, its kind, the tiles left of
        // that kind, and where its tokens (l0 .. l0 + 31 of the batch row) begin in the tensor of that kind.  (Worked out per tile it was
        // half of the tile's instructions.)
        const unsigned char* st = s_w;
        int ring = NS;
        int kind = kind0, kind_left = kind_left0;
        bf16_t* to = PROJ ? a.q + row_base + (size_t)l0 * a.D + to0
                          : a.out + (size_t)(((int64_t)(a.r0 + rl) * a.sr + (int64_t)l0 * a.sl) * a.N + ft_begin * 32);
        for (int n = 0; n < n_ft; ++n) {
            const int ft = ft_begin + n;
            if (run) {
                f32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0.f;
                uint32_t pk[8];
                // (opaque and fenced: else the operand addresses of all steps, and all operands, are in registers at once, and others in scratch memory)
                unsigned rd = rd0;
                asm volatile("" : "+v"(rd));
                auto contract = [&](auto&& mac) __attribute__((always_inline)) {
                    constexpr int AHEAD = KC >= 16 ? 3 : (KC < 4 ? KC : 4);              // operand reads in flight
                    Frag wf[AHEAD];
#pragma unroll
                    for (int s = 0; s < AHEAD; ++s) wf[s].u = *reinterpret_cast<const uint4*>(st + (rd ^ (32u * s)));
#pragma unroll
                    for (int s = 0; s < KC; ++s) {
                        mac(s, wf[s % AHEAD]);
                        if (s + AHEAD < KC) wf[s % AHEAD].u = *reinterpret_cast<const uint4*>(st + (rd ^ (32u * (s + AHEAD))));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (PROJ && kind == TK_V) {
                    // lane = feature, value v = token 8 (v / 4) + 4 hf + v % 4
                    contract([&](int s, const Frag& w) __attribute__((always_inline)) { acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[s].v, w.v, acc, 0, 0, 0); });
                    Frag wx;
                    wx.u = s_aug[n * 32 + col];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xaug.v, wx.v, acc, 0, 0, 0);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float4 rs = *reinterpret_cast<const float4*>(s_rstd + wave * 32 + 8 * g + 4 * hf);
                        pk[2 * g] = pack2(acc[4 * g] * rs.x, acc[4 * g + 1] * rs.y);
                        pk[2 * g + 1] = pack2(acc[4 * g + 2] * rs.z, acc[4 * g + 3] * rs.w);
                    }
                } else {
                    // lane = token, value v = feature 8 (v / 4) + 4 hf + v % 4
                    contract([&](int s, const Frag& w) __attribute__((always_inline)) { acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.v, xa[s].v, acc, 0, 0, 0); });
                    if constexpr (PROJ) {
                        Frag wx;
                        wx.u = s_aug[n * 32 + col];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wx.v, xaug.v, acc, 0, 0, 0);
                    }
                    if constexpr (RES) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sel[0].v, rn[0].v, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sel[1].v, rn[1].v, acc, 0, 0, 0);
                        load_res(ft + 1);
                        n_ops += 2;
                    }
                    if constexpr (!PROJ) {
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const float4 c = *reinterpret_cast<const float4*>(s_cn + n * 32 + 8 * g + 4 * hf);
                            pk[2 * g] = pack2(acc[4 * g] + c.x, acc[4 * g + 1] + c.y);
                            pk[2 * g + 1] = pack2(acc[4 * g + 2] + c.z, acc[4 * g + 3] + c.w);
                        }
                    } else if (kind == TK_GATE) {
                        const float nr = -kLog2e * rstd;
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            pk[i] = pack2(__builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc[2 * i] * nr)),
                                          __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc[2 * i + 1] * nr)));
                    } else if (kind == TK_BIAS) {
                        // pair bias: feature = head, token (rl, l) = pair (q, k)
                        int lq = l;
                        asm volatile("" : "+v"(lq));                           // (the sixteen addresses: not before the loop)
                        float* bp = a.bias + bias_index(4 * hf, a.r0 + rl, lq, a.Lq, a.Lp);
                        int plane = a.Lq * a.Lp;
                        asm volatile("" : "+s"(plane));                        // (and the sixteen multiples of it)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int hu = 8 * (v >> 2) + (v & 3);               // head of the lower half-wave
                            if (hu < a.H - 4 * hf) bp[(size_t)hu * plane] = acc[v] * rstd;
                        }
                        continue;                                              // (the last tile)
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) pk[i] = pack2(acc[2 * i] * rstd, acc[2 * i + 1] * rstd);
                    }
                }
                // A lane holds the 16-byte pieces hf and 2 + hf of its token's (v: feature's) 64 bytes.  Where these are 64 bytes of memory too
                // they are exchanged so that the first store has all four pieces of the first sixteen tokens, piece 2 (row % 2) + row / 2 in
                // the row of sixteen lanes, and the second those of the others: each writes whole 64-byte rows (halves of 32 rows: 42 us instead of
                // 38 for the projections of 64 x 2048 tokens).
                merge_halves(pk[0], pk[2]);
                merge_halves(pk[1], pk[3]);
                merge_halves(pk[4], pk[6]);
                merge_halves(pk[5], pk[7]);
                if (!PROJ || kind == TK_V || a.D == 32)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto sw = __builtin_amdgcn_permlane16_swap(pk[i], pk[4 + i], false, false);
                    pk[i] = sw[0];
                    pk[4 + i] = sw[1];
                }
                const uint4 lo = make_uint4(pk[0], pk[1], pk[2], pk[3]), hi = make_uint4(pk[4], pk[5], pk[6], pk[7]);
                if constexpr (PROJ) {
                    // q, k, gate: [row][head][l][d]; v^T tiled by 32 keys: [row][head][l / 32][e][l % 32].  One place for all of them: of two
                    // the compiler merges the ends, and writes the second store in pieces of 4 and 12 bytes
                    const unsigned at = kind == TK_V ? v_lane : t_lane;
                    *reinterpret_cast<uint4*>(to + at) = lo;
                    *reinterpret_cast<uint4*>(to + at + (kind == TK_V ? v_second : t_second)) = hi;
                    n_ops += 2;
                } else {                                           // out: [token][N]
                    if (l0 + (lane & 15) < a.L) *reinterpret_cast<uint4*>(to + o_lane) = lo;
                    if (l0 + 16 + (lane & 15) < a.L) *reinterpret_cast<uint4*>(to + o_lane + 16 * a.sl * a.N) = hi;
                    if (l0 < a.L) n_ops += l0 + 16 < a.L ? 2 : 1;  // (wave-uniform: the instructions were issued)
                }
            }
            st = st + STAGE < s_w + 2 * NS * STAGE ? st + STAGE : s_w;
            if constexpr (PROJ) {
                to += tile_step;
                if (--kind_left == 0) {
                    asm volatile("");                         // (a branch: seldom taken)
                    ++kind;
                    kind_left = per_kind;
                    to += (kind == TK_V ? 2 : (kind == TK_GATE ? -1 : 1)) * a.tensor - a.H * LpD;      // (q, k, gate, v^T)
                }
            } else {
                to += 32;
            }
            if (--ring == 0 && !whole && n + 1 < n_ft) {
                ring = NS;
                // Order of this wavefront's memory operations: ... L(i+1), S, L(i+2), S, ... (L = loads of a half, S = the stores
                // issued during one half).  The next half needs L(i+1): everything but the stores issued after it must have completed.
                // After the barrier all wavefronts have their share of L(i+1) in LDS and have finished
                // reading this half, which the loads of the half after next then overwrite.
                wait_vmem_but_last(__builtin_amdgcn_readfirstlane(n_ops));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                n_ops = 0;
                const int next = n + 1 + NS;
                if (next < n_ft) issue(next, n_ft - next < NS ? n_ft - next : NS, next % (2 * NS));
            }
        }
        if (!whole) break;
        unit += a.along * NW;
        if (unit >= tiles_m) break;
    }
}

// ====================================================================================
// Projection and attention in one kernel, for sequences of at most 256 positions with head
// dimension 32 (the row-wise and triangle attentions of the training crop, Section 5.2's merged
// projections feeding its fused softmax): a block takes two batch rows and one head, projects
// that head's q, k, v and gate for all tokens of the two rows straight from the raw input (the
// LayerNorm folded into the weights as in k_gemm) and attends at once.  q and the gate never
// leave the registers, k and v^T live in LDS, so that of the five tensors k_gemm<PROJ> hands to
// the attention kernel through HBM only the gated context is ever written.
//
// Wavefront w owns tokens 32w .. 32w+31 of both rows: as projection tokens first, as queries
// afterwards.  A projection tile leaves the matrix core with the lane = token, register =
// feature 8*(v/4) + 4*hf + v%4 layout; packed in register order it is a valid B operand of
// S^T = K Q^T as long as the key side uses the same order of the contraction, which is how the k
// tile is written to LDS (one 16-byte piece per step and half-wave).  The gate has the layout
// of O^T already.  v is computed with the operands swapped (lane = feature), which is the
// layout of a row of v^T.  The bias tile of a key tile is loaded once and used as accumulator
// input for both rows.
//
// LDS: the head's four folded 32 x K weight tiles (row pitch 2K + 16 bytes), their extra pieces,
// k [2][256][80 bytes], v^T [2][32][528 bytes], 1/std of the tokens, one word per (row, key tile) with a bit per
// valid key, and 2 KiB per wavefront through which the raw tokens, fetched as
// whole 128-byte lines, are turned into matrix-core operands.  With 256 channels that is 159 KiB
// of the compute unit's 160: one block of eight wavefronts per compute unit.
//
// The attention phase is the pipeline of k_attn_rows over two rows: no reference in the softmax, masked keys cost a matrix
// instruction only in tiles that hold any, matrix instructions of the next and the previous tile between the exponentials.
//
// Measured on the training crop of the row-wise attention (128 x 256 tokens, 8 heads): 41 to 43 us under the profiler, where k_gemm<PROJ> and an attention kernel took
// 34 + 31; triangle attention at 256: 34 to 36.  In the projections a weight operand is read from LDS once for the tokens of both rows, three steps ahead (one
// read per instruction, waited for: 62.7 us the call instead of 62.3, no more than the runs of one side differ); of the two wavefronts of a SIMD
// the older one is served first and finishes each phase about a quarter earlier, and the block waits for the younger one
// at both barriers.

struct FusedArgs {
    const bf16_t* x;       // raw input, token (r, l) at (r*sr + l*sl)*K
    int64_t sr, sl;        // token strides of x and of the mask
    int r0, rows, L, Lp, Lq;
    float eps;
    const bf16_t* wp;      // prepared weights [(4*Hd + 32)][K]
    const uint4* aug;      // their extra pieces
    int H, Hd;
    const float* bias;     // tiled (bias_index) or NULL
    const float* mask;     // caller's mask or NULL
    bf16_t* o;             // gated context [rows][H][Lp][32]
};

constexpr int kFuKPitch = 80;       // bytes of a key row in LDS (64 and a pad: conflict-free operand reads)
constexpr int kFuVPitch = 528;      // bytes of a v^T row in LDS: 256 keys and a pad
constexpr int kFuWaves = 8;

static size_t fused_smem_bytes(int kc) {
    return (size_t)4 * 32 * (32 * kc + 16) + 128 * 16 + 2 * 256 * kFuKPitch + 2 * 32 * kFuVPitch + kFuWaves * 2 * 32 * 4 + 64 +
           kFuWaves * 2048;
}

template <int KC, bool HAS_BIAS>
__global__ __launch_bounds__(kFuWaves * 64) void k_proj_attn(FusedArgs a) {
    constexpr int K = 16 * KC, WP = 32 * KC + 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* s_w = smem;                                                  // [4][32][WP]
    uint4* s_aug = reinterpret_cast<uint4*>(s_w + 4 * 32 * WP);                 // [4][32]
    unsigned char* s_k = reinterpret_cast<unsigned char*>(s_aug + 128);         // [2][256][kFuKPitch]
    unsigned char* s_vt = s_k + 2 * 256 * kFuKPitch;                            // [2][32][kFuVPitch]
    float* s_stat = reinterpret_cast<float*>(s_vt + 2 * 32 * kFuVPitch);        // [wave][2][32]
    int* s_live = reinterpret_cast<int*>(s_stat + kFuWaves * 2 * 32);           // [2][8]: bit = key of the tile is attended to
    unsigned char* s_st = reinterpret_cast<unsigned char*>(s_live + 16) + (threadIdx.x >> 6) * 2048;   // [wave][16][128]

    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = a.Lp >> 5;                               // 32-token tiles of a row, at most 8
    const bool active = wave < nt;                          // (wave-uniform)
    // Work-groups go to the 8 XCDs round-robin and each XCD has its own L2: the heads of a row
    // pair run on one XCD at about the same time, so the rows of x come from HBM once.  Item
    // jj*H + h of an XCD is row pair xcd + 8 jj, head h; a block takes the items slot, slot +
    // slots, ...: with the slots a multiple of H its head never changes and the weights are
    // loaded once.
    const int n_rp = (a.rows + 1) >> 1;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
    const int n_local = xcd < n_rp ? ((n_rp - xcd + 7) >> 3) * a.H : 0;
    int h_loaded = -1;
    // the lane's index formed anew, where an address made of it would otherwise be held through the whole item: at 256 channels it was held in scratch memory, and
    // fetched from there behind every load in flight
    auto fresh_lane = []() __attribute__((always_inline)) {
        int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(l));
        return l;
    };
    const int l_tok = 32 * wave + col;
    const bool tok_in = active && l_tok < a.L;
    const bool has_mask = a.mask != nullptr;

    for (int it = slot; it < n_local; it += slots) {
        const int jj = it / a.H, h = it - jj * a.H;
        const int rp = xcd + 8 * jj;
        // ---- raw tokens (row 0 issued first; row 1 follows line by line as the registers fall free),
        // the mask entries.  Eight lanes fetch one 128-byte line of a token (a load with lane =
        // token, the operand layout, touches 64 lines for 1 KiB and the cache looks up one line per
        // cycle: 5 us per item instead of 1.2; no load is under a condition, each a branch of its own); raw[m][hh][i] holds line m of the tokens 16hh + 8i +
        // lane/8 of the wavefront's tile, piece lane%8.  Issued before the barrier: the loads are on
        // their way while the block waits for its last wavefront.
        constexpr int NG = KC / 4;              // 128-byte lines per token
        uint4 raw[NG][2][2];
        float mval[2];
        bool row_ok[2];
        int rlv[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int rl = 2 * rp + j;
            row_ok[j] = rl < a.rows;
            rlv[j] = row_ok[j] ? rl : a.rows - 1;
            mval[j] = 1.f;
            if (has_mask && tok_in) mval[j] = a.mask[(int64_t)(a.r0 + rlv[j]) * a.sr + (int64_t)l_tok * a.sl];
        }
        auto fetch_line = [&](int j, int m) __attribute__((always_inline)) {
            const int64_t row_tok = (int64_t)(a.r0 + rlv[j]) * a.sr;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int l = 32 * wave + 16 * hh + 8 * i + (lane >> 3);
                    raw[m][hh][i] = ldg16(a.x + (row_tok + (int64_t)(l < a.L ? l : a.L - 1) * a.sl) * K + (lane & 7) * 8 + 64 * m);
                }
        };
#pragma unroll
        for (int m = 0; m < NG; ++m) fetch_line(0, m);

        if (it != slot) __syncthreads();            // every wavefront has left the item before: k and v^T may be overwritten

        // ---- the head's weight tiles
        if (h != h_loaded) {
            // (128 rows of 2 KC pieces, KC / 2 pieces per thread, up to four loads in flight)
            constexpr int WB = KC / 2 < 4 ? KC / 2 : 4;          // loads in flight per thread
            const int t = 64 * wave + fresh_lane();
#pragma unroll
            for (int n0 = 0; n0 < KC / 2; n0 += WB) {
                uint4 wv[WB];
#pragma unroll
                for (int n = 0; n < WB; ++n) {
                    const int p = t + (n0 + n) * kFuWaves * 64;
                    const int row = p / (2 * KC), pp = p - row * (2 * KC);
                    wv[n] = ldg16(a.wp + ((size_t)((row >> 5) * a.Hd + h * 32 + (row & 31)) * K + pp * 8));
                }
#pragma unroll
                for (int n = 0; n < WB; ++n) {
                    const int p = t + (n0 + n) * kFuWaves * 64;
                    const int row = p / (2 * KC), pp = p - row * (2 * KC);
                    *reinterpret_cast<uint4*>(s_w + row * WP + pp * 16) = wv[n];
                }
            }
            if (t < 128) s_aug[t] = a.aug[(t >> 5) * a.Hd + h * 32 + (t & 31)];
            h_loaded = h;
            __syncthreads();
        }

        // ---- projections: q and gate stay in registers, k and v^T go to LDS
        Frag qf[2][2];          // (set and used by wavefronts with tokens only)
        uint32_t gpk[2][8];
        if (active) {
            // ---- both rows' tokens as operands, with their statistics
            Frag xa[2][KC], xaug[2];
            float rstd[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                // The lines pass through the wavefront's staging area (16 tokens x 128 bytes, the eight
                // pieces of a token rotated by its index: conflict-free) and come back in the operand
                // layout, lane = token, pieces 2s' + hf of line m = contraction steps 4m + s'.  The
                // area is private to the wavefront, whose LDS operations complete in order.
                float sum = 0.f, sq = 0.f;
#pragma unroll
                for (int m = 0; m < NG; ++m) {
                    Frag* xg = &xa[j][4 * m];
                    // (defined anew, with whatever the registers hold: each half of the lanes is loaded under a condition below, and the compiler would keep
                    // the last item's operands through the attention for the other half)
#pragma unroll
                    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
                        for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(xg[sp].w[i]));
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const int tl = 8 * i + (lane >> 3);
                            *reinterpret_cast<uint4*>(s_st + tl * 128 + (((lane & 7) ^ (tl & 7)) * 16)) = raw[m][hh][i];
                        }
                        __builtin_amdgcn_wave_barrier();
                        if ((col >> 4) == hh) {
                            const int tl = col & 15;
#pragma unroll
                            for (int sp = 0; sp < 4; ++sp)
                                xg[sp].u = *reinterpret_cast<const uint4*>(s_st + tl * 128 + (((2 * sp + hf) ^ (tl & 7)) * 16));
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                    if (j == 0) fetch_line(1, m);         // (the line's registers are free again)
                    if (32 * wave + 32 > a.L) {           // (wave-uniform; tokens beyond L hold the last one: they must not bring its infinities or NaN to the keys)
                        const uint32_t keep = l_tok < a.L ? 0xffffffffu : 0u;
#pragma unroll
                        for (int sp = 0; sp < 4; ++sp)
                            xg[sp].u = make_uint4(xg[sp].u.x & keep, xg[sp].u.y & keep, xg[sp].u.z & keep, xg[sp].u.w & keep);
                    }
                    // LayerNorm statistics as in token_stats, one line at a time
#pragma unroll
                    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            sum = add_pair(xg[sp].w[i], sum);
                            sq = add_pair_sq(xg[sp].w[i], sq);
                        }
                }
                sum += other_half(sum);
                sq += other_half(sq);
                const float mu = sum * (1.f / (float)K);
                const float var = fmaxf(sq * (1.f / (float)K) - mu * mu, 0.f) + a.eps;
                rstd[j] = tok_in ? rsqrtf(var) : 0.f;
                const float mneg = tok_in ? -mu : 0.f, r = var * rstd[j];
                const float m_hi = bf16_round(mneg), m_lo = bf16_round(mneg - m_hi);
                const float r_hi = bf16_round(r), r_lo = bf16_round(r - r_hi);
                xaug[j].u = make_uint4(0, 0, 0, 0);
                if (hf == 0) {
                    xaug[j].u = make_uint4(pack2(m_hi, m_hi), pack2(m_lo, r_hi), pack2(r_hi, r_lo), 0u);
                    s_stat[(wave * 2 + j) * 32 + (fresh_lane() & 31)] = rstd[j];
                }
                const bool key_valid = tok_in && mval[j] != 0.f;
                const uint64_t live = __ballot(key_valid);           // (the two half-waves hold the same 32 tokens)
                if (lane == 0) s_live[j * 8 + wave] = (int)(uint32_t)live;
            }
            // ---- the head's four feature tiles one after the other, every weight operand read from LDS once for the tokens of both rows
            f32x16 acc[2];
            auto contract = [&](int T, bool tokens_first) __attribute__((always_inline)) {
                // (opaque and fenced: else the operands of all steps are in registers at once, and others in scratch memory)
                unsigned rd = (unsigned)(T * 32 * WP + col * WP + hf * 16);
                asm volatile("" : "+v"(rd));
                constexpr int AHEAD = 3;
                Frag wf[AHEAD];
#pragma unroll
                for (int st = 0; st < AHEAD; ++st) wf[st].u = *reinterpret_cast<const uint4*>(s_w + (rd + 32u * st));
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
#pragma unroll
                for (int st = 0; st <= KC; ++st) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const Frag& x = st < KC ? xa[j][st < KC ? st : 0] : xaug[j];
                        acc[j] = tokens_first ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, wf[st % AHEAD].v, acc[j], 0, 0, 0)
                                              : __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[st % AHEAD].v, x.v, acc[j], 0, 0, 0);
                    }
                    if (st + AHEAD < KC) wf[st % AHEAD].u = *reinterpret_cast<const uint4*>(s_w + (rd + 32u * (st + AHEAD)));
                    else if (st + AHEAD == KC) wf[st % AHEAD].u = s_aug[32 * T + col];
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // k: one 16-byte piece per step and half-wave into the token's LDS row
            contract(1, false);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                unsigned char* krow = s_k + (j * 256 + l_tok) * kFuKPitch;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    uint32_t kw[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) kw[i] = pack2(acc[j][8 * s + 2 * i] * rstd[j], acc[j][8 * s + 2 * i + 1] * rstd[j]);
                    *reinterpret_cast<uint4*>(krow + (2 * s + hf) * 16) = make_uint4(kw[0], kw[1], kw[2], kw[3]);
                }
            }
            // v: lane = feature col, register v = token 8*(v/4) + 4*hf + v%4 of the wavefront's tile
            // (1/std of those tokens comes back from LDS: written above by this wavefront, whose LDS
            // operations complete in order)
            contract(2, true);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                unsigned char* vrow = s_vt + (j * 32 + col) * kFuVPitch + (32 * wave + 4 * hf) * 2;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 rs = *reinterpret_cast<const float4*>(s_stat + (wave * 2 + j) * 32 + 8 * g + 4 * hf);
                    *reinterpret_cast<uint2*>(vrow + 16 * g) = make_uint2(pack2(acc[j][4 * g] * rs.x, acc[j][4 * g + 1] * rs.y),
                                                                          pack2(acc[j][4 * g + 2] * rs.z, acc[j][4 * g + 3] * rs.w));
                }
            }
            // q: B operand of S^T, step s = registers 8s .. 8s+7, the order of k's pieces
            contract(0, false);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) qf[j][i >> 2].w[i & 3] = pack2(acc[j][2 * i] * rstd[j], acc[j][2 * i + 1] * rstd[j]);
            // gate: the layout of O^T
            contract(3, false);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float nr = -kLog2e * rstd[j];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    gpk[j][i] = pack2(__builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc[j][2 * i] * nr)),
                                      __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(acc[j][2 * i + 1] * nr)));
            }
        }
        __syncthreads();

        // ---- attention of the wavefront's 32 queries of both rows over the nt key tiles
        if (active) {
            // (the lane's indices anew, opaque to the optimiser: the addresses of this phase would
            // otherwise be computed before the projections and held in registers through them)
            int lane_a = lane;
            asm volatile("" : "+v"(lane_a));
            const int col_a = lane_a & 31, hf_a = lane_a >> 5;
            // permuted key of S^T row m = col: rows 8g + 4b + e hold key 16*(g/2) + 8b + 4*(g%2) + e, so that the lane's registers 8c .. 8c+7 hold
            // the keys 16c + 8hf .. + 7 of the tile
            const int kperm_a = 16 * (col_a >> 4) + 8 * ((col_a >> 2) & 1) + 4 * ((col_a >> 3) & 1) + (col_a & 3);
            int nk = 1;                                       // key tiles up to the last one with a valid key in either row
            for (int t = 1; t < nt; ++t)
                if (__builtin_amdgcn_readfirstlane(s_live[t] | s_live[8 + t]) != 0) nk = t + 1;
            f32x16 o_acc[2], s_acc[2];
            float l_run[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                l_run[j] = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) o_acc[j][v] = 0.f;
            }
            // (tiled bias, see bias_index: the tiles of the wavefront's 32 queries follow each other)
            const float* bh = HAS_BIAS ? a.bias + ((size_t)h * (a.Lq >> 5) + wave) * nt * 1024 : nullptr;
            // (the lane of a query beyond L takes the last real one's: nobody has written its own, and the denominators multiply its weights by zero)
            const int last_q = a.L - 1 - 32 * wave;
            const uint32_t b_lane = (uint32_t)((col_a < last_q ? col_a : last_q) + 32 * hf_a) * 16;
            auto load_bias = [&](int kt, f32x16& bt) __attribute__((always_inline)) {
                if constexpr (HAS_BIAS) {
                    if (kt > nk - 1) kt = nk - 1;             // (past the end: a harmless repeat)
                    const char* bp = reinterpret_cast<const char*>(bh + 1024 * kt) + b_lane;
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const float4 x4 = *reinterpret_cast<const float4*>(bp + (2 * c + i) * 1024);
                            bt[8 * c + 4 * i] = x4.x; bt[8 * c + 4 * i + 1] = x4.y;
                            bt[8 * c + 4 * i + 2] = x4.z; bt[8 * c + 4 * i + 3] = x4.w;
                        }
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v) bt[v] = 0.f;
                }
            };
            const uint32_t k_lane = (uint32_t)(kperm_a * kFuKPitch + hf_a * 16), v_lane = (uint32_t)(col_a * kFuVPitch + 16 * hf_a);
            auto load_k = [&](int j, int kt, Frag (&kf)[2]) __attribute__((always_inline)) {
                if (kt > nk - 1) kt = nk - 1;
                const unsigned char* kr = s_k + (j * 256 + 32 * kt) * kFuKPitch + k_lane;
                kf[0].u = *reinterpret_cast<const uint4*>(kr);
                kf[1].u = *reinterpret_cast<const uint4*>(kr + 32);
            };
            auto load_v = [&](int j, int kt, Frag (&vf)[2]) __attribute__((always_inline)) {
                const unsigned char* vr = s_vt + j * 32 * kFuVPitch + 64 * kt + v_lane;
                vf[0].u = *reinterpret_cast<const uint4*>(vr);
                vf[1].u = *reinterpret_cast<const uint4*>(vr + 32);
            };
            Frag kf[2][2], vf[2][2], pf[2];
            const bf16x8 sel = sum_select(lane_a);
#pragma unroll
            for (int c = 0; c < 2; ++c) pf[c].u = vf[1][c].u = make_uint4(0, 0, 0, 0);
            // The pipeline of k_attn_rows over the tiles (kt, row 0), (kt, row 1), ...: the exponentials of a tile run while the
            // matrix core forms the scores of the next one (bias bn, keys live_n) and the context and the denominator of the one before
            auto tile = [&](uint32_t live_n, f32x16& sc, f32x16& sn, const f32x16& bn, Frag (&qn)[2], Frag (&kn)[2], Frag (&vp)[2],
                            f32x16& op, float& lp, auto&& loads) __attribute__((always_inline)) {
                Frag pc[2];
                f32x4 lt = {0.f, 0.f, 0.f, 0.f};
                float e0 = __builtin_amdgcn_exp2f(sc[0]), e1 = __builtin_amdgcn_exp2f(sc[1]);
#pragma unroll
                for (int g = 0; g < 8; ++g) {
                    if (g == 0) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kn[0].v, qn[0].v, bn, 0, 0, 0);
                    if (g == 2) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kn[1].v, qn[1].v, sn, 0, 0, 0);
                    if (g == 4) op = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp[0].v, pf[0].v, op, 0, 0, 0);
                    if (g == 6) op = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp[1].v, pf[1].v, op, 0, 0, 0);
                    if (g == 4 && live_n != 0xffffffffu) sn = mask_step(live_n, kperm_a, hf_a, sn);
                    if ((g & 3) == 3) lt = add_piece(sel, pf[g >> 2].v, lt);
                    if (g == 0) loads();
                    float n0 = 0.f, n1 = 0.f;
                    if (g < 7) {
                        n0 = __builtin_amdgcn_exp2f(sc[2 * g + 2]);
                        n1 = __builtin_amdgcn_exp2f(sc[2 * g + 3]);
                        asm volatile("" : "+v"(n0), "+v"(n1));
                    }
                    uint32_t& w = pc[g >> 2].w[g & 3];
                    w = pack2(e0, e1);
                    asm volatile("" : "+v"(w));
                    __builtin_amdgcn_sched_barrier(0);
                    e0 = n0;
                    e1 = n1;
                }
                lp += lt[0];
                pf[0] = pc[0];
                pf[1] = pc[1];
            };
            auto live_of = [&](int j, int kt) __attribute__((always_inline)) {
                return (uint32_t)__builtin_amdgcn_readfirstlane(s_live[j * 8 + (kt < nk ? kt : nk - 1)]);
            };
            auto step = [&](int kt, f32x16& bc, f32x16& bn) __attribute__((always_inline)) {
                const uint32_t l1 = live_of(1, kt), l0 = live_of(0, kt + 1);
                tile(l1, s_acc[0], s_acc[1], bc, qf[1], kf[1], vf[1], o_acc[1], l_run[1], [&]() __attribute__((always_inline)) {
                    load_k(0, kt + 1, kf[0]);
                    load_v(0, kt, vf[0]);
                });
                tile(l0, s_acc[1], s_acc[0], bn, qf[0], kf[0], vf[0], o_acc[0], l_run[0], [&]() __attribute__((always_inline)) {
                    load_k(1, kt + 1, kf[1]);
                    load_v(1, kt, vf[1]);
                    load_bias(kt + 2, bc);
                });
            };
            f32x16 bA, bB;
            load_bias(0, bA);
            load_bias(1, bB);
            load_k(0, 0, kf[0]);
            load_k(1, 0, kf[1]);
            s_acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][0].v, qf[0][0].v, bA, 0, 0, 0);
            s_acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][1].v, qf[0][1].v, s_acc[0], 0, 0, 0);
            s_acc[0] = mask_step(live_of(0, 0), kperm_a, hf_a, s_acc[0]);
            int kt = 0;
            for (; kt + 1 < nk; kt += 2) {
                step(kt, bA, bB);
                step(kt + 1, bB, bA);
            }
            if (kt < nk) step(kt, bA, bB);
            {
                f32x4 lt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    o_acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[1][c].v, pf[c].v, o_acc[1], 0, 0, 0);
                    lt = add_piece(sel, pf[c].v, lt);
                }
                l_run[1] += lt[0];
            }
            // rows that do not stand are done again with a running maximum
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (!__any(!softmax_stands<16>(o_acc[j], l_run[j]) && l_tok < a.L)) continue;
                float m = -INFINITY;
                l_run[j] = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) o_acc[j][v] = 0.f;
                for (int t = 0; t < nk; ++t) {
                    const uint32_t live = live_of(j, t);
                    if (live == 0) continue;
                    f32x16 s;
                    load_bias(t, s);
                    load_k(j, t, kf[0]);
                    load_v(j, t, vf[0]);
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][0].v, qf[j][0].v, s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][1].v, qf[j][1].v, s, 0, 0, 0);
                    general_tile(s, vf[0], live, hf_a, o_acc[j], m, l_run[j]);
                }
                l_run[j] += other_half(l_run[j]);
            }

            // ---- normalise, gate, store: o_acc[j]: lane = query, register v = e = 8*(v/4) + 4*hf + v%4
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float l_tot = l_run[j];
                const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
                uint32_t pk[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    pk[i] = pack2(o_acc[j][2 * i] * inv * lo_f32(gpk[j][i]), o_acc[j][2 * i + 1] * inv * hi_f32(gpk[j][i]));
                merge_halves(pk[0], pk[2]);      // lower half-wave: e 0..7, upper: e 8..15
                merge_halves(pk[1], pk[3]);
                merge_halves(pk[4], pk[6]);      // lower: e 16..23, upper: e 24..31
                merge_halves(pk[5], pk[7]);
                bf16_t* op = a.o + ((size_t)(rlv[j] * a.H + h) * a.Lp + 32 * wave) * 32;        // (uniform)
                const int ln = fresh_lane();
                const uint32_t o_lane = (uint32_t)((ln & 31) * 32 + 8 * (ln >> 5)) * 2;
                if (row_ok[j] && 32 * wave + (ln & 31) < a.L) {
                    stg16(op, o_lane, make_uint4(pk[0], pk[1], pk[2], pk[3]));
                    stg16(op + 16, o_lane, make_uint4(pk[4], pk[5], pk[6], pk[7]));
                }
            }
        }
    }
}

// ====================================================================================
// host side
// More than 64 KiB of dynamic LDS has to be asked for once per kernel.  The request is the
// initialiser of a function-local static: the language runs it exactly once, also when several
// threads make their first call together, and every caller sees its result.
template <typename Kernel>
static hipError_t allow_large_lds(Kernel kernel) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               96 * 1024);
}

template <int KC, bool PROJ, bool RES>
static ff_status launch_gemm_inst(GemmArgs a, int tiles_m, hipStream_t st) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm<KC, PROJ, RES>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return fail(FF_EHIP, "k_gemm: dynamic LDS limit: %s", hipGetErrorString(attr));
    // Blocks of eight wavefronts or of all that a compute unit holds, one token tile each, and the feature tiles shared out over `split` such blocks: what
    // makes the rounds of blocks times the time of a block least.  A block takes its tiles and about five more for its tokens and first
    // weights, each the longer the more wavefronts its compute unit really holds (fewer than fit where the grid does not fill the chip), and a seventh
    // more through the ring with its barriers.  The constants lie where the regret over all splits of 160 launches is least (both kernels of 94 calls from
    // 8 x 48 to 2048 x 2048 tokens, 32 to 256 channels): 0.2 % of the call on average and 4 % at most above the best split, 93 % of
    // them within 1 %.  (Charging every block for the wavefronts that could share its unit, ten tiles and 24 wavefronts: 1.2 % on average, 11 % at most -
    // twelve wavefronts for the outputs of 32 x 64 tokens of 256 channels, 27.1 us the call, eight 25.4; projections of 384 x 384 tokens
    // in 288 blocks, two rounds, 161.5, in two shares 149.)
    const int cu = compute_units();
    a.waves = 8;
    double least = 1e300;
    constexpr bool large_first = KC > 4;                     // (of equals the larger blocks, which load the weights less often; where those are short the smaller ones)
    for (int nw : {large_first ? gemm_waves(KC) : 8, large_first ? 8 : gemm_waves(KC)}) {
        const int along = (tiles_m + nw - 1) / nw;
        for (int t = 1, next; t <= a.ft_count; t = t < a.ft_count && next > a.ft_count ? a.ft_count : next) {
            next = t + (t < 8 ? 1 : t / 4);
            const int per = (a.ft_count + t - 1) / t, n = (a.ft_count + per - 1) / per;
            // (65 to 128 channels: more than 22 tiles with their offsets and extra pieces do not fit beside the ring)
            // (nor, at any size that memory holds, more blocks than split_inv divides exactly)
            if (gemm_smem_bytes(KC, per) > 160 * 1024 || (n > 1 && (int64_t)along * n * n >= ((int64_t)1 << 31))) continue;
            // blocks per compute unit (gemm_fit: what the registers allow)
            const int fit = 2 * nw <= gemm_fit(KC, PROJ) && 2 * gemm_smem_bytes(KC, per) <= 160 * 1024 ? 2 : 1;
            const double blocks = (double)along * n;
            const bool whole = per <= 2 * gemm_half(KC);
            const double cost = ceil(blocks / (cu * fit)) * (5 + per) * (8 + nw * fmin(fit, ceil(blocks / cu))) * (whole ? 1 : 1.15);
            if (cost >= least) continue;
            least = cost;
            // (whole weights: no more blocks than are resident, each takes more tokens)
            a.along = whole && blocks > cu * fit ? (cu * fit + n - 1) / n : along;
            a.split = n; a.tiles_per_split = per;
            a.waves = nw;
        }
    }
    a.split_inv = a.split > 1 ? (uint32_t)((((uint64_t)1 << 32) + a.split - 1) / a.split) : 0u;
    a.per_xcd = (a.along * a.split + 7) / 8;
    hipLaunchKernelGGL((k_gemm<KC, PROJ, RES>), dim3(8 * a.per_xcd), dim3(a.waves * 64), gemm_smem_bytes(KC, a.tiles_per_split), st, a);
    return FF_OK;
}

template <bool PROJ, bool RES>
static ff_status launch_gemm(const GemmArgs& a, hipStream_t st) {
    const int tiles_m = a.rows * (a.Lp >> 5);
    if (a.K <= 32) return launch_gemm_inst<2, PROJ, RES>(a, tiles_m, st);
    if (a.K <= 64) return launch_gemm_inst<4, PROJ, RES>(a, tiles_m, st);
    if (a.K <= 128) return launch_gemm_inst<8, PROJ, RES>(a, tiles_m, st);
    return launch_gemm_inst<16, PROJ, RES>(a, tiles_m, st);
}

// Units of 64 queries of one head of eight batch rows (of four without a bias, where a wavefront takes two rows, and in small chunks): a unit has at
// most 512 threads of k_attn_rows' grid (attn_rows_launch: blocks of two wavefronts and two rows up to two tiles, else of four wavefronts
// and four rows, two without a bias) and 512 padded tokens of one head, so below 2^22 units both are less than 2^31, and the kernels count both in an int.
constexpr int chunk_unit_rows(bool small, bool bias) { return small || !bias ? 4 : 8; }
constexpr bool unit_holds_512_threads(bool bias) {
    for (int nt = 1; nt <= 16384 / 32; ++nt) {
        const int waves = nt <= 2 ? 2 : 4, rows = nt <= 2 || !bias ? 2 : 4, rb = chunk_unit_rows(false, bias);
        if ((nt + waves - 1) / waves * ((rb + rows - 1) / rows) * waves * 64 > 512 * ((nt + 1) / 2)) return false;
    }
    return true;
}
static_assert(unit_holds_512_threads(true) && unit_holds_512_threads(false), "the limit of mfma_chunk_ok covers the grid of k_attn_rows");
bool mfma_chunk_ok(const Problem& p, int chunk) {
    const int rb = chunk_unit_rows(chunk < 8, p.has_bias);
    return (int64_t)(round_up(p.L, 64) / 64) * p.H * ((chunk + rb - 1) / rb) < (1 << 22);
}

static int query_compute_units() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
        return v;
    return 256;
}
// (queried once; a function-local static is initialised exactly once, also under concurrent first calls)
int compute_units() {
    static const int n = query_compute_units();
    return n;
}

static bool fused_proj_attn(const Problem& p);

static GemmArgs proj_args(const Problem& p, const MfmaWs& m, const Workspace& ws) {
    const int Lp = round_up(p.L, 32), Lq = round_up(p.L, 32);
    GemmArgs g{};
    g.sr = p.sr; g.sl = p.sl; g.L = p.L; g.Lp = Lp; g.Lq = Lq; g.K = p.c; g.eps = p.eps;
    g.w = m.wp; g.aug = m.aug; g.Hd = p.Hd; g.H = p.H; g.D = p.d; g.dsh = p.d == 8 ? 3 : (p.d == 16 ? 4 : 5);
    g.nt_main = 4 * p.Hd / 32;
    g.q = m.q; g.tensor = m.k - m.q; g.bias = ws.bias;
    return g;
}

ff_status mfma_prepare(const Problem& p, const ff_attn_weights& w, const void* x, const void* z, const Workspace& ws,
                       hipStream_t st) {
    const MfmaWs m = split_ws(p, ws.chunk, ws);
    const int Lp = round_up(p.L, 32), Lq = round_up(p.L, 32);
    const float qscale = kLog2e / sqrtf((float)p.d);
    const bool tri = p.mode == FF_TRI_START || p.mode == FF_TRI_END;
    {
        const bf16_t *gm = (const bf16_t*)w.ln_g, *bt = (const bf16_t*)w.ln_b;
        const int Hd = p.Hd, c = p.c;
        PrepArgs a{};
        auto seg = [&](int i, const void* wsrc, const void* extra, int rows, int rows_pad, int row0, float scale) {
            a.seg[i] = {(const bf16_t*)wsrc, (const bf16_t*)extra, gm, bt, m.wp + (size_t)row0 * c, m.aug + row0,
                        rows, rows_pad, c, scale};
        };
        seg(0, w.w_q, nullptr, Hd, Hd, 0, qscale);
        seg(1, w.w_k, nullptr, Hd, Hd, Hd, 1.f);
        seg(2, w.w_v, nullptr, Hd, Hd, 2 * Hd, 1.f);
        seg(3, w.w_g, w.b_g, Hd, Hd, 3 * Hd, 1.f);
        seg(4, tri ? w.w_b : nullptr, nullptr, tri ? p.H : 0, 32, 4 * Hd, kLog2e);
        a.nseg = 5;
        const int rows = 4 * Hd + 32;
        const bool chunked_tri = tri && (ws.chunk < p.R || (p.has_bias && fused_proj_attn(p)));
        if (p.mode == FF_MSA_ROW || chunked_tri) {
            // the pair-bias pass shares the launch: row mode projects z (own LayerNorm); chunked
            // triangle attention needs the bias of all rows before the first chunk
            PrepBiasArgs b{};
            b.prep = a;
            b.bias_blocks = (p.L * (Lp / 32) + 7) / 8;
            b.w_b = (const bf16_t*)w.w_b;
            if (chunked_tri) {
                b.z = (const bf16_t*)x; b.sr = p.sr; b.sl = p.sl; b.K = p.c;
                b.gamma = gm; b.beta = bt;
            } else {
                b.z = (const bf16_t*)z; b.sr = p.L; b.sl = 1; b.K = p.c_z;
                b.gamma = (const bf16_t*)w.lnz_g; b.beta = (const bf16_t*)w.lnz_b;
            }
            b.bias = ws.bias; b.L = p.L; b.Lp = Lp; b.Lq = Lq; b.H = p.H; b.eps = p.eps;
            const dim3 grid(b.bias_blocks + (rows + 7) / 8);
            const int kc = (b.K + 15) / 16;
            Timed t(KK_BIAS, st);
            if (kc <= 2) hipLaunchKernelGGL(k_prep_bias<2>, grid, dim3(512), 0, st, b);
            else if (kc <= 4) hipLaunchKernelGGL(k_prep_bias<4>, grid, dim3(512), 0, st, b);
            else if (kc <= 8) hipLaunchKernelGGL(k_prep_bias<8>, grid, dim3(512), 0, st, b);
            else hipLaunchKernelGGL(k_prep_bias<16>, grid, dim3(512), 0, st, b);
        } else {
            Timed t(KK_PREP, st);
            hipLaunchKernelGGL(k_prep, dim3((rows + 3) / 4), dim3(256), 0, st, a);
        }
    }
    return check_launch("prepare (mfma)");
}

// Shapes that k_proj_attn takes: head dimension 32, between 129 and 256 positions (fewer would leave
// most of its eight wavefronts without tokens), 64, 128 or 256 channels.  The pair bias then comes
// from k_prep_bias in every mode (the triangle modes too: it cannot ride along with projections
// that never leave the attention kernel), in the tiled layout of bias_index.
static bool fused_proj_attn(const Problem& p) {
    if (p.d != 32 || p.L <= 128 || p.L > 256) return false;
    return p.c == 64 || p.c == 128 || p.c == 256;
}

template <int KC, bool HAS_BIAS>
static ff_status launch_fused(const FusedArgs& a, hipStream_t st) {
    static const hipError_t attr = allow_large_lds(&k_proj_attn<KC, HAS_BIAS>);
    if (attr != hipSuccess) return fail(FF_EHIP, "k_proj_attn: dynamic LDS limit: %s", hipGetErrorString(attr));
    // one block per compute unit (LDS); per XCD at most as many blocks as it has items
    const int n_rp = (a.rows + 1) / 2;
    int slots = compute_units() / 8;
    const int items_xcd = ((n_rp + 7) / 8) * a.H;
    if (slots > items_xcd) slots = items_xcd;
    if (slots < 1) slots = 1;
    hipLaunchKernelGGL((k_proj_attn<KC, HAS_BIAS>), dim3(8 * slots), dim3(kFuWaves * 64), fused_smem_bytes(KC), st, a);
    return FF_OK;
}

ff_status mfma_chunk(const Problem& p, const ff_attn_weights& w, const void* x, const float* mask, const void* res,
                     void* out, const Workspace& ws, int r0, int rows, hipStream_t st) {
    const int Lp = round_up(p.L, 32), Lq = round_up(p.L, 32);
    const MfmaWs m = split_ws(p, ws.chunk, ws);
    const bool tri = p.mode == FF_TRI_START || p.mode == FF_TRI_END;
    const bool fused = fused_proj_attn(p);
    if (fused) {
        FusedArgs f{};
        f.x = (const bf16_t*)x; f.sr = p.sr; f.sl = p.sl; f.r0 = r0; f.rows = rows; f.L = p.L; f.Lp = Lp; f.Lq = Lq;
        f.eps = p.eps; f.wp = m.wp; f.aug = m.aug; f.H = p.H; f.Hd = p.Hd; f.bias = ws.bias; f.mask = mask; f.o = m.o;
        Timed t(KK_PROJ_ATTN, st);
        ff_status ls = FF_OK;
#define FF_FUSED(KCV)                                              \
    do {                                                           \
        if (p.has_bias) ls = launch_fused<KCV, true>(f, st);       \
        else ls = launch_fused<KCV, false>(f, st);                 \
    } while (0)
        if (p.c == 64) FF_FUSED(4);
        else if (p.c == 128) FF_FUSED(8);
        else FF_FUSED(16);
#undef FF_FUSED
        if (ls != FF_OK) return ls;
    } else {
        GemmArgs g = proj_args(p, m, ws);
        g.src = (const bf16_t*)x; g.r0 = r0; g.rows = rows;
        // one chunk covering every row: the pair-bias tile rides along with the projections
        const bool fused_bias = tri && ws.chunk >= p.R;
        g.ft_count = g.nt_main + (fused_bias ? 1 : 0);
        Timed t(KK_PROJ, st);
        const ff_status ls = launch_gemm<true, false>(g, st);
        if (ls != FF_OK) return ls;
    }

    if (!fused) {
        AttnRowsArgs r{};
        r.q = m.q; r.k = m.k; r.g = m.g; r.vt = m.vt; r.o = m.o; r.bias = ws.bias; r.mask = mask;
        r.sr = p.sr; r.sl = p.sl; r.r0 = r0; r.rows = rows; r.L = p.L; r.Lp = Lp; r.Lq = Lq; r.H = p.H;
        Timed t(KK_ATTN, st);
        const ff_status ls = attn_rows_launch(r, p.d, st);
        if (ls != FF_OK) return ls;
    }

    GemmArgs o{};
    o.src = m.o; o.sr = p.sr; o.sl = p.sl; o.r0 = r0; o.rows = rows; o.L = p.L; o.Lp = Lp; o.Lq = Lq;
    o.K = p.Hd; o.w = (const bf16_t*)w.w_o; o.bvec = (const bf16_t*)w.b_o;
    o.Hd = p.Hd; o.H = p.H; o.D = p.d; o.dsh = p.d == 8 ? 3 : (p.d == 16 ? 4 : 5); o.out = (bf16_t*)out; o.N = p.c;
    o.odd_step = p.d == 32 ? 16 : Lp * 16; o.even_step = p.d == 32 ? Lp * 32 - 16 : o.odd_step;
    {
        o.ft_count = o.N / 32;
        Timed t(KK_OUT, st);
        o.res = (const bf16_t*)res;
        const ff_status ls = res ? launch_gemm<false, true>(o, st) : launch_gemm<false, false>(o, st);
        if (ls != FF_OK) return ls;
    }
    return check_launch("attention chunk (mfma)");
}

}  // namespace ff
