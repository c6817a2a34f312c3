// Backward pass of the fused attention core (FastFold Section 6.3 benchmarks the fused softmax forward and
// backward; Table 6 reports forward and backward per Evoformer layer), bf16 operands, float32 statistics and
// accumulators, gfx950 matrix cores.  Per batch row r and head h, with scale = 1 / sqrt(d):
//   S[i,j] = scale q[i].k[j] + bias[h,i,j] + M(mask[r,j]);  P = softmax_j S;  ctx[i] = sum_j P[i,j] v[j];  o = g * ctx
//   dg = do * ctx;  dctx = do * g;  dv[j] = sum_i P[i,j] dctx[i];  dP[i,j] = dctx[i].v[j];
//   dS[i,j] = P[i,j] (dP[i,j] - delta[i]),  delta[i] = dctx[i].ctx[i];
//   dq[i] = scale sum_j dS[i,j] k[j];  dk[j] = scale sum_i dS[i,j] q[i];  dbias[h,i,j] = sum_r dS[r,h,i,j]
//
// The score matrix is never stored (Section 3.2): as in the forward pass it is recomputed tile by tile.
// Launches:
//   k_bwd_prepare  the bias times sqrt(d), tile by tile in the order of the accumulator registers, once with lane = query and
//                once with lane = key, so that a bias tile is four 16-byte loads per lane in every kernel; the key masks as bits
//   k_bwd_rows   up to 512 positions of enough (row, head)s (rows_in_lds): a block per (row, head), everything but the bias gradient:
//                forward recomputation with an online softmax (the logsumexp of every query, base 2, ctx, dg and delta), then P and dS once
//                for dq, dk and dv
//   k_bwd_stats, k_bwd_dq, k_bwd_dkv   longer sequences, and few (row, head)s of more than 320 positions: the same in three kernels, one wavefront per 32-query (or 32-key) tile, four
//                consecutive tiles of one (row, head) per block; the tiles of the other side, which all four contract with, are copied into LDS
//                once per block, a tile ahead of the arithmetic.  dq: S^T = K Q^T and dP^T = V dctx^T (lane = query, so that
//                logsumexp and delta are lane-local), dS^T, dq^T += K^T dS^T; dkv: S = Q K^T and dP = dctx V^T (lane = key), P and
//                dS, dv^T += dctx^T P, dk^T += Q^T dS
//   k_bwd_dbias  per (head, patch of 4 x 4 tiles, chunk of batch rows): dS summed in registers over the rows of the
//                chunk, the chunks' partial sums added in a fixed order by a small second kernel (deterministic,
//                no atomics)
// Operands whose contraction runs over the head dim are 16-byte row reads of the staged tiles; operands whose contraction
// runs over keys or queries (lane = channel) are transposing reads of the same tiles (ds_read_b64_tr_b16: no
// position-contiguous copy of any tensor exists), taken in exactly the order in which the accumulator of the previous
// contraction leaves its values, so
// nothing moves between two contractions.  What is added to q.k and what is subtracted from dP enter through the
// matrix core: the bias tile and -delta as the accumulators' starting values, the -inf of masked keys as one more
// contraction step (key side 0 or -inf, query side 1).  A thread's share of the staging copies (which pieces,
// from where, to where) is worked out once per block (StagePlan), not per tile.
// Operand layouts of v_mfma_f32_32x32x16_bf16: A (32 x 16): lane l holds row l%32, columns 8*(l/32)..+7;
// B (16 x 32): lane l holds column l%32, rows 8*(l/32)..+7; D (32 x 32): lane l holds column l%32, register
// v holds row 8*(v/4) + 4*(l/32) + v%4.
#include "ff_common.h"

namespace ff {
namespace bwd {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

union Frag {
    bf16x8 v;
    uint4 u;
    uint32_t w[4];
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    bf16x2 t;
    t[0] = (__bf16)a;
    t[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, t);
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

static inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

struct Args {
    const bf16_t *q, *k, *v, *g, *dout;      // [R][H][L][D]
    const float* bias;                       // [H][L][L] or NULL
    const float* mask;                       // [R][L] or NULL
    const float* mrow;                       // mask entry of (r, j): mrow[r * mstride + j] (without a mask: a row of ones, stride 0)
    int mstride;
    float* ones;                             // workspace [Lp]: that row of ones (written by k_bwd_prepare)
    bf16_t *dq, *dk, *dv, *dg;               // [R][H][L][D]
    float* dbias;                            // [H][L][L] or NULL
    float* dbias_part;                       // workspace [row_chunks][H][Lp/32][Lp/32][4][64][4]: partial sums over the rows of a chunk, ordered as biasA
    int row_chunks, rows_per_chunk;
    bf16_t* dctx;                            // workspace [R][H][L][D]
    float *lse, *delta;                      // workspace [R*H][2][Lp]: logsumexp and delta of a (row, head) side by side (delta = lse + Lp)
    uint32_t* live;                          // workspace [R][Lp/32]: bit = key is attended to (written by k_bwd_prepare when there is a bias)
    float *biasA, *biasK;                    // workspace [H][Lp/32][Lp/32][4][64][4]: the bias, times sqrt(D), tile by tile in the
                                             // order of the accumulator registers (biasA: lane = query, biasK: lane = key)
    int R, H, L, Lp;
    float qscale2;                           // log2(e) / sqrt(D)
    float scale;                             // 1 / sqrt(D)
    float sqrt_d;                            // sqrt(D)
};

// Row fragments of the 32 positions n0 .. n0+31 of x [L][D] (x already offset to its (row, head)): lane (n, hf)
// holds channels 16 s + 8 hf .. + 7 of position n0 + col; zeros beyond L or D.
template <int D, bool FULL = false>       // FULL: the caller knows n0 + 31 < L
__device__ __forceinline__ void load_rows(Frag (&f)[(D + 15) / 16], const bf16_t* x, int n0, int L, int col, int hf) {
    constexpr int KS = (D + 15) / 16;
    const int n = n0 + col;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        f[s].u = make_uint4(0, 0, 0, 0);
        if ((FULL || n < L) && 16 * s + 8 * hf < D) f[s].u = *reinterpret_cast<const uint4*>(x + (size_t)n * D + 16 * s + 8 * hf);
    }
}

// The tiled copies of the bias (see Args) and the row of ones.  One wavefront per 32 x 32 tile of a head.
__global__ __launch_bounds__(256) void k_bwd_prepare(Args a) {
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = a.Lp >> 5;
    if (blockIdx.x == 0)
        for (int n = threadIdx.x; n < a.Lp; n += 256) a.ones[n] = 1.f;
    const int task = blockIdx.x * 4 + wave;
    if (!a.bias) return;
    if (task >= a.H * nt * nt) {                     // the wavefronts behind the tiles: the key masks of two tiles of a batch row as bits
        const int pairs = (nt + 1) >> 1, w = task - a.H * nt * nt;
        const int r = w / pairs, jt = 2 * (w - r * pairs), j = 32 * jt + lane;
        if (r >= a.R) return;
        const uint64_t bits = __ballot(j < a.L && (a.mask == nullptr || a.mask[(size_t)r * a.L + (j < a.L ? j : 0)] != 0.f));
        if (lane == 0) a.live[(size_t)r * nt + jt] = (uint32_t)bits;
        if (lane == 0 && jt + 1 < nt) a.live[(size_t)r * nt + jt + 1] = (uint32_t)(bits >> 32);
        return;
    }
    // The bias tile (it, jt) of head h, times sqrt(D), as the accumulator of the logits holds it: float4 g of
    // lane (col, hf) = entries 8 g + 4 hf .. + 3 along the register axis.  biasK: lane = key j0 + col, registers
    // along the queries, as the rows are read (128 bytes of a row per half-wave); biasA: lane = query i0 + col, registers along the
    // keys, through the wavefront's own LDS tile.  Zeros outside [0, L)^2.
    __shared__ float s_t[4][32 * 33];
    const int h = task / (nt * nt), rem = task - h * nt * nt, it = rem / nt, jt = rem - it * nt;
    const float* bh = a.bias + (size_t)h * a.L * a.L;
    float* ta = a.biasA + (size_t)task * 1024 + lane * 4;
    float* tk = a.biasK + (size_t)task * 1024 + lane * 4;
    float* t = s_t[wave];
    float vk[16];
    const int j = jt * 32 + col, jc = j < a.L ? j : a.L - 1;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int i = it * 32 + 8 * (v >> 2) + 4 * hf + (v & 3);
        const float x = bh[(size_t)(i < a.L ? i : a.L - 1) * a.L + jc];
        vk[v] = i < a.L && j < a.L ? x * a.sqrt_d : 0.f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) t[(8 * (v >> 2) + 4 * hf + (v & 3)) * 33 + col] = vk[v];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        *reinterpret_cast<float4*>(tk + 256 * g) = make_float4(vk[4 * g], vk[4 * g + 1], vk[4 * g + 2], vk[4 * g + 3]);
        const float* u = t + col * 33 + 8 * g + 4 * hf;
        *reinterpret_cast<float4*>(ta + 256 * g) = make_float4(u[0], u[1], u[2], u[3]);
    }
}

// registers 8s .. 8s+7 of an accumulator, rounded to bf16: the B operand of contraction step s over its rows
__device__ __forceinline__ void pack_rows(Frag (&f)[2], const f32x16& a) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) f[s].w[i] = pack2(a[8 * s + 2 * i], a[8 * s + 2 * i + 1]);
}

__device__ __forceinline__ f32x16 zero16() {
    f32x16 a;
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] = 0.f;
    return a;
}

// The logits enter the matrix core's accumulator already holding what is added to q.k: S = (q.k + B) * scale with
// B[i][j] = bias[h][i][j] * sqrt(d) for a key that may be attended to and -inf for one that is masked or beyond L
// (exp2 of the base-2 logit then gives weight 0 without any select).  The bias part comes from the copies that
// k_bwd_prepare leaves in the order of the accumulator registers (four 16-byte loads per lane and tile, a
// contiguous KiB per instruction; bias_tile_fetch can run tiles ahead).  The -inf part is one more matrix
// instruction: a contraction step whose key side holds 0 or -inf in its first slot and whose query side a one.
__device__ __forceinline__ void bias_tile_fetch(float4 (&rows)[4], const float* tiles, int h, int nt, int it, int jt, int lane) {
    const char* p = reinterpret_cast<const char*>(tiles + (((size_t)h * nt + it) * nt + jt) * 1024);     // (uniform)
    const uint32_t off = (uint32_t)lane * 16;
#pragma unroll
    for (int g = 0; g < 4; ++g) rows[g] = *reinterpret_cast<const float4*>(p + 1024 * g + off);
}
__device__ __forceinline__ void rows_to_acc(f32x16& b, const float4 (&rows)[4]) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        b[4 * g] = rows[g].x; b[4 * g + 1] = rows[g].y; b[4 * g + 2] = rows[g].z; b[4 * g + 3] = rows[g].w;
    }
}
// operand fragments of that step: ok = the lane's key may be attended to
__device__ __forceinline__ Frag key_side(bool ok, int hf) {
    Frag f;
    f.u = make_uint4((hf == 0 && !ok) ? 0xff80u : 0u, 0u, 0u, 0u);        // bfloat16 -inf
    return f;
}
__device__ __forceinline__ Frag one_side(int hf) {
    Frag f;
    f.u = make_uint4(hf == 0 ? 0x3f80u : 0u, 0u, 0u, 0u);                 // bfloat16 1
    return f;
}

// ====================================================================================
// Staging of a 32-position tile of one (row, head) for the four wavefronts of a block, which all contract with it:
// the row-major tile of two tensors (x, y: [32][D]) and two float vectors of the 32 positions.  The block copies 16-byte
// pieces global -> registers -> LDS, one tile ahead of the tile being worked on (two LDS stages, one barrier per tile); a
// wavefront reads its operand fragments from LDS just before the matrix instructions that use them.
constexpr int kStPitch = 80;                          // bytes per staged row: 32 bf16 + 16 bytes, 16-byte aligned
constexpr int kStRowsX = 0, kStRowsY = 32 * kStPitch;
constexpr int kStVecA = 64 * kStPitch, kStVecB = kStVecA + 128, kStSpare = kStVecB + 128, kStBytes = kStSpare + 16;

struct TileSrc {
    const bf16_t *x, *y;         // [L][D] of the (row, head)
    const float *va, *vb;        // [Lp] of the (row, head), or NULL
    int L, Lp;
};

// A thread moves up to two 16-byte pieces of every tile.  Which pieces, where they come from and where they go in the
// stage does not depend on the tile, so it is worked out once (StagePlan::init): per piece the address for tile
// position 0, the bytes per position and the offset in the stage.  A piece nobody needs (its vector is NULL, or the
// thread has no second piece) asks for the start of x again and lands in a spare slot of the stage: every load and
// every store of the loop is unconditional.
template <int D, bool FULL>
struct StagePlan {
    const unsigned char *b0, *b1;          // piece address at tile position 0
    int s0, s1;                            // bytes per position
    int d0, d1;                            // offset in the stage
    int n0_, n1_;                          // !FULL: position of a row piece within the tile (zeros beyond L), else a large negative number

    static __device__ __forceinline__ void piece(const TileSrc& t, int id, const unsigned char*& base, int& stride, int& dst, int& row) {
        constexpr int PR = D / 8, NR = 32 * PR, N = 2 * NR + 16;
        static_assert(N <= 512, "two pieces per thread");
        base = reinterpret_cast<const unsigned char*>(t.x); stride = 0; dst = kStSpare; row = -(1 << 30);
        if (id >= N) return;
        if (id < 2 * NR) {
            const bool second = id >= NR;
            const int k = second ? id - NR : id, n = k / PR, pc = k - n * PR;
            const bf16_t* src = second ? t.y : t.x;
            base = reinterpret_cast<const unsigned char*>(src + (size_t)n * D + 8 * pc); stride = 2 * D;
            dst = (second ? kStRowsY : kStRowsX) + n * kStPitch + pc * 16; row = n;
            return;
        }
        id -= 2 * NR;
        const bool second = id >= 8;
        const int pc = second ? id - 8 : id;
        const float* src = second ? t.vb : t.va;
        if (!src) return;
        base = reinterpret_cast<const unsigned char*>(src + 4 * pc); stride = 4;
        dst = (second ? kStVecB : kStVecA) + pc * 16;
    }
    __device__ __forceinline__ void init(const TileSrc& t, int tid) {
        piece(t, tid, b0, s0, d0, n0_);
        piece(t, tid + 256, b1, s1, d1, n1_);
    }
    // the pieces of the tile at position n: requested from memory (rows at positions >= L: the last one again) ...
    __device__ __forceinline__ void fetch(int n, int L, uint4& r0, uint4& r1) const {
        const int m0 = FULL || n < L - n0_ ? n : L - 1 - n0_, m1 = FULL || n < L - n1_ ? n : L - 1 - n1_;
        r0 = *reinterpret_cast<const uint4*>(b0 + (int64_t)m0 * s0);
        r1 = *reinterpret_cast<const uint4*>(b1 + (int64_t)m1 * s1);
    }
    // ... and put into the stage (L: rows at positions n + row >= L are zeros)
    __device__ __forceinline__ void store(unsigned char* stage, int n, int L, uint4 r0, uint4 r1) const {
        const uint4 z = make_uint4(0, 0, 0, 0);
        if (!FULL) {
            if (n + n0_ >= L) r0 = z;
            if (n + n1_ >= L) r1 = z;
        }
        *reinterpret_cast<uint4*>(stage + d0) = r0;
        *reinterpret_cast<uint4*>(stage + d1) = r1;
    }
};
// operand fragments out of a stage: rows of the lane's position (as load_rows), channels of the lane (below)
template <int D>
__device__ __forceinline__ void staged_rows(Frag (&f)[(D + 15) / 16], const unsigned char* rows, int col, int hf) {
#pragma unroll
    for (int s = 0; s < (D + 15) / 16; ++s) {
        f[s].u = make_uint4(0, 0, 0, 0);
        if (16 * s + 8 * hf < D) f[s].u = *reinterpret_cast<const uint4*>(rows + col * kStPitch + (16 * s + 8 * hf) * 2);
    }
}
// Lane (e, hf) gets x[n][e] for the eight positions that slot u = 0..7 of half hf of contraction step s meets, n = 16 s + 4 hf +
// (u < 4 ? u : u + 4): the order in which a 32 x 32 accumulator (register 8s + u of half hf) leaves its rows.  Two
// transposing 8-byte reads per step: of sixteen lanes, lane i asks for four channels 4 (i % 4) .. of position i / 4, and lane l
// receives channel l of the four positions.  Lanes of channels beyond D receive what the rows' padding holds; it reaches only rows
// of the result that nobody stores.
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef __attribute__((address_space(3))) i16x4* lds_i16x4;
__device__ __forceinline__ void staged_cols(Frag (&f)[2], const unsigned char* rows, int lane) {
    const unsigned char* p = rows + (4 * (lane >> 5) + ((lane >> 2) & 3)) * kStPitch + ((lane & 16) + 4 * (lane & 3)) * 2;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)(p + 16 * s * kStPitch)));
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)(p + (16 * s + 8) * kStPitch)));
        f[s].u = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
}

// Rows of masked keys in a stage become zeros: their weights are zero, but zero times a NaN is not.  Every wavefront does so for itself before it
// reads (its LDS operations complete in order, and the others write the same zeros), and only in tiles that hold masked keys, which it knows
// before the barrier in front of the tile.  (Dropped on their way into the stage, every tile waited for its mask entries: 2 to 5 % of a call
// of few (row, head)s.)
template <int D>
__device__ __forceinline__ void zero_masked(unsigned char* stage, bool ok, int col, int hf) {
    if (ok) return;
#pragma unroll
    for (int pc = 0; pc < D / 8; pc += 2)
        if (pc + hf < D / 8) {
            *reinterpret_cast<uint4*>(stage + kStRowsX + col * kStPitch + (pc + hf) * 16) = make_uint4(0, 0, 0, 0);
            *reinterpret_cast<uint4*>(stage + kStRowsY + col * kStPitch + (pc + hf) * 16) = make_uint4(0, 0, 0, 0);
        }
}

// Tile loop of the two kernels whose wavefronts keep a query tile and walk over the key tiles.  Memory is one
// tile ahead of the arithmetic: while tile t is worked on, tile t + 1 is being requested, and it goes into the free LDS stage at
// the end of tile t.  Two named register sets (even tiles, odd
// tiles), hence a loop body written for a literal parity P and used twice: tile tt + P, stage P, sets [P].
//   rs[P]: staged pieces of the thread; brow[P]: the lane's bias rows; mk[P]: the lane's key-mask entry.
#define FF_BWD_Q_PROLOGUE                                                                                        \
    uint4 rs[2][2];                                                                                              \
    float4 brow[2][4];                                                                                           \
    float mk[2] = {1.f, 1.f};                                                                                    \
    const int i0a = active ? i0 : 0;                                                                             \
    const float* mrow = a.mrow + (size_t)r * a.mstride;                                                          \
    plan.fetch(0, a.L, rs[0][0], rs[0][1]);                                                                      \
    if (BIAS) bias_tile_fetch(brow[0], a.biasA, h, nt, i0a >> 5, 0, lane);                                       \
    if (FULL || col < a.L) mk[0] = mrow[col];                                                                    \
    plan.store(s_stage, 0, a.L, rs[0][0], rs[0][1]);                                                             \
    bool masked = !__all((FULL || col < a.L) && mk[0] != 0.f);           /* the tile in the stage holds masked keys */ \
    __syncthreads();
// (bt and kx: what the accumulator of the logits starts from, see bias_tile_fetch.  Every load of the loop is issued on
// every path - the last tile asks for itself again - because a load under a condition makes the compiler
// wait, at every later wait, also for the loads just issued.)
#define FF_BWD_Q_HEAD(P)                                                                                         \
    const int j0 = 32 * (tt + (P));                                                                              \
    unsigned char* stage = s_stage + (P) * kStBytes;                                                             \
    constexpr int PF = 1 - (P);                           /* the register set that receives what is requested now */ \
    const int jn = j0 + 32 < a.L ? j0 + 32 : j0;                                                                 \
    plan.fetch(jn, a.L, rs[PF][0], rs[PF][1]);                                                                   \
    const bool key_ok = (FULL || j0 + col < a.L) && mk[P] != 0.f;                                                \
    const Frag kx = key_side(key_ok, hf);                                                                        \
    if (masked) zero_masked<D>(stage, key_ok, col, hf);                                                          \
    f32x16 bt;                                                                                                   \
    if (BIAS) rows_to_acc(bt, brow[P]);                                                                          \
    else bt = zero16();                                                                                          \
    if (BIAS) bias_tile_fetch(brow[PF], a.biasA, h, nt, i0a >> 5, jn >> 5, lane);                                \
    if (FULL || jn + col < a.L) mk[PF] = mrow[jn + col];
#define FF_BWD_Q_TAIL(P)                                                                                         \
    if (j0 + 32 < a.L)                                                                                           \
        plan.store(s_stage + (1 - (P)) * kStBytes, j0 + 32, a.L, rs[1 - (P)][0], rs[1 - (P)][1]);                \
    masked = !__all((FULL || j0 + 32 + col < a.L) && mk[1 - (P)] != 0.f);                                        \
    __syncthreads();

// ====================================================================================
// Block = four consecutive query tiles of one (row, head); the key-side tiles (k and v rows) are
// staged once per block and key tile; the bias rows and the key-mask entries of the next tile are requested
// while this one is worked on.
template <int D, bool FULL, bool BIAS>
__global__ __launch_bounds__(256) void k_bwd_stats(Args a) {
    constexpr int KS = (D + 15) / 16;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[2 * kStBytes];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = a.Lp >> 5, bpr = (nt + 3) >> 2;
    const int rh = blockIdx.x / bpr, it = (blockIdx.x - rh * bpr) * 4 + wave;
    const int r = rh / a.H, h = rh - r * a.H, i0 = it * 32, i = i0 + col;
    const bool active = it < nt;
    const size_t base = (size_t)rh * a.L * D;
    TileSrc src;
    src.x = a.k + base; src.y = a.v + base;
    src.va = nullptr; src.vb = nullptr; src.L = a.L; src.Lp = a.Lp;
    Frag qf[KS];
    load_rows<D, FULL>(qf, a.q + base, active ? i0 : 0, a.L, col, hf);
    StagePlan<D, FULL> plan;
    plan.init(src, tid);
    FF_BWD_Q_PROLOGUE
    const Frag one = one_side(hf);

    // (the reference starts finite: exp2(-inf - m) is 0 for a masked key, not NaN, also before the first valid one)
    constexpr float kSlack = 8.f;
    float m = -1e30f, l = 0.f;
    f32x16 ctx = zero16();          // ctx^T: lane = query, register v = channel 8(v/4) + 4hf + v%4
#define FF_BWD_STATS_TILE(P)                                                                                     \
    {                                                                                                            \
        FF_BWD_Q_HEAD(P)                                                                                         \
        if (active) {                                                                                            \
            Frag kf[KS], vt[2], pf[2];                                                                           \
            staged_rows<D>(kf, stage + kStRowsX, col, hf);                                                       \
            staged_cols(vt, stage + kStRowsY, lane);                                                             \
            f32x16 s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx.v, one.v, bt, 0, 0, 0);                        \
            _Pragma("unroll") for (int t = 0; t < KS; ++t)                                                       \
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t].v, qf[t].v, s, 0, 0, 0);                       \
            float tmax = s[0];                                                                                   \
            _Pragma("unroll") for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);                             \
            tmax *= a.qscale2;                                      /* (qscale2 > 0) */                          \
            /* m is the query's reference for the exponentials (the same in its two lanes), not its exact       \
               maximum: it moves, and the sums are rescaled, only when a logit of the tile exceeds it by more    \
               than kSlack - after a query's first tiles almost never, and then the tile pays neither for the    \
               exchange between the halves nor for the rescaling; weights stay below 2^kSlack */                 \
            if (__builtin_amdgcn_ballot_w64(tmax > m + kSlack) != 0) {                                           \
                const float m_new = fmaxf(m, half_max(tmax));                                     \
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);                                           \
                _Pragma("unroll") for (int v = 0; v < 16; ++v) ctx[v] *= alpha;                                  \
                l *= alpha;                                                                                      \
                m = m_new;                                                                                       \
            }                                                                                                    \
            float lt = 0.f;                                                                                      \
            _Pragma("unroll") for (int v = 0; v < 16; ++v) {                                                     \
                s[v] = __builtin_amdgcn_exp2f(s[v] * a.qscale2 - m);                                             \
                lt += s[v];                                                                                      \
            }                                                                                                    \
            l += lt;                                                                                             \
            pack_rows(pf, s);                                                                                    \
            _Pragma("unroll") for (int t = 0; t < 2; ++t)                                                        \
                ctx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt[t].v, pf[t].v, ctx, 0, 0, 0);                   \
        }                                                                                                        \
        FF_BWD_Q_TAIL(P)                                                                                         \
    }
    for (int tt = 0; 32 * tt < a.L; tt += 2) {
        FF_BWD_STATS_TILE(0)
        if (32 * (tt + 1) < a.L) FF_BWD_STATS_TILE(1)
    }
#undef FF_BWD_STATS_TILE
    if (!active) return;             // (no barrier after this point)
    const float l_tot = half_sum(l);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    // a query without unmasked keys: logsumexp = +inf makes every recomputed weight exp2(s - inf) = 0
    const float lse = l_tot > 0.f ? m + __builtin_amdgcn_logf(l_tot) : INFINITY;

    float dl = 0.f;
    if (i < a.L) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const int e0 = 8 * gq + 4 * hf;
            if (e0 < D) {
                const size_t off = base + (size_t)i * D + e0;
                const uint2 dov = *reinterpret_cast<const uint2*>(a.dout + off);
                const uint2 gv = *reinterpret_cast<const uint2*>(a.g + off);
                const float d_o[4] = {lo_f32(dov.x), hi_f32(dov.x), lo_f32(dov.y), hi_f32(dov.y)};
                const float gg[4] = {lo_f32(gv.x), hi_f32(gv.x), lo_f32(gv.y), hi_f32(gv.y)};
                float dgv[4], dc[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float c = ctx[4 * gq + e] * inv;
                    dgv[e] = d_o[e] * c;
                    // delta uses the very dctx values the other kernels read (rounded to bf16)
                    dc[e] = lo_f32(pack2(d_o[e] * gg[e], 0.f));
                    dl += dc[e] * c;
                }
                *reinterpret_cast<uint2*>(a.dg + off) = make_uint2(pack2(dgv[0], dgv[1]), pack2(dgv[2], dgv[3]));
                *reinterpret_cast<uint2*>(a.dctx + off) = make_uint2(pack2(dc[0], dc[1]), pack2(dc[2], dc[3]));
            }
        }
    }
    dl = half_sum(dl);
    if (hf == 0) {       // (Lp slots per (row, head): queries beyond L get a defined value too)
        a.lse[(size_t)rh * 2 * a.Lp + i] = i < a.L ? lse : INFINITY;
        a.delta[(size_t)rh * 2 * a.Lp + i] = dl;
    }
}

// ====================================================================================
// Block = four consecutive query tiles of one (row, head); staged per key tile: k rows and v rows.
template <int D, bool FULL, bool BIAS>
__global__ __launch_bounds__(256, 3) void k_bwd_dq(Args a) {
    constexpr int KS = (D + 15) / 16;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[2 * kStBytes];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = a.Lp >> 5, bpr = (nt + 3) >> 2;
    const int rh = blockIdx.x / bpr, it = (blockIdx.x - rh * bpr) * 4 + wave;
    const int r = rh / a.H, h = rh - r * a.H, i0 = it * 32, i = i0 + col;
    const bool active = it < nt;
    const size_t base = (size_t)rh * a.L * D;
    TileSrc src;
    src.x = a.k + base; src.y = a.v + base;
    src.va = nullptr; src.vb = nullptr; src.L = a.L; src.Lp = a.Lp;
    Frag qf[KS], dcf[KS];
    load_rows<D, FULL>(qf, a.q + base, active ? i0 : 0, a.L, col, hf);
    load_rows<D, FULL>(dcf, a.dctx + base, active ? i0 : 0, a.L, col, hf);
    const float lse = a.lse[(size_t)rh * 2 * a.Lp + (active ? i : col)], delta = a.delta[(size_t)rh * 2 * a.Lp + (active ? i : col)];
    StagePlan<D, FULL> plan;
    plan.init(src, tid);
    FF_BWD_Q_PROLOGUE
    const Frag one = one_side(hf);

    f32x16 dq = zero16();           // dq^T: lane = query, register = channel
    f32x16 ndelta;
#pragma unroll
    for (int v = 0; v < 16; ++v) ndelta[v] = -delta;
#define FF_BWD_DQ_TILE(P)                                                                                        \
    {                                                                                                            \
        FF_BWD_Q_HEAD(P)                                                                                         \
        if (active) {                                                                                            \
            Frag kf[KS], vf[KS], kt[2], dsf[2];                                                                  \
            staged_rows<D>(kf, stage + kStRowsX, col, hf);                                                       \
            staged_rows<D>(vf, stage + kStRowsY, col, hf);                                                       \
            f32x16 s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx.v, one.v, bt, 0, 0, 0);                        \
            f32x16 dp = ndelta;              /* dP - delta: the accumulator starts from -delta */                \
            _Pragma("unroll") for (int t = 0; t < KS; ++t) {                                                     \
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t].v, qf[t].v, s, 0, 0, 0);                       \
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t].v, dcf[t].v, dp, 0, 0, 0);                    \
            }                                                                                                    \
            staged_cols(kt, stage + kStRowsX, lane);                                                             \
            _Pragma("unroll") for (int v = 0; v < 16; ++v)                                                       \
                s[v] = __builtin_amdgcn_exp2f(s[v] * a.qscale2 - lse) * dp[v];                                   \
            pack_rows(dsf, s);                                                                                   \
            _Pragma("unroll") for (int t = 0; t < 2; ++t)                                                        \
                dq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[t].v, dsf[t].v, dq, 0, 0, 0);                    \
        }                                                                                                        \
        FF_BWD_Q_TAIL(P)                                                                                         \
    }
    for (int tt = 0; 32 * tt < a.L; tt += 2) {
        FF_BWD_DQ_TILE(0)
        if (32 * (tt + 1) < a.L) FF_BWD_DQ_TILE(1)
    }
#undef FF_BWD_DQ_TILE
    if (active && i < a.L) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const int e0 = 8 * gq + 4 * hf;
            if (e0 < D)
                *reinterpret_cast<uint2*>(a.dq + base + (size_t)i * D + e0) =
                    make_uint2(pack2(dq[4 * gq] * a.scale, dq[4 * gq + 1] * a.scale),
                               pack2(dq[4 * gq + 2] * a.scale, dq[4 * gq + 3] * a.scale));
        }
    }
}

// ====================================================================================
// Block = four consecutive key tiles of one (row, head); the query-side tiles (q, dctx, logsumexp,
// delta) are staged once per block and query tile.
// (three wavefronts per SIMD where the lengths are whole tiles: at d = 32 with a bias that costs four spilled
// registers, all outside the tile loop; in the variant with bounds checks one of them would land inside it, and a
// reload inside the loop is waited for together with every load in flight)
template <int D, bool FULL, bool BIAS>
__global__ __launch_bounds__(256, FULL ? 3 : 1) void k_bwd_dkv(Args a) {
    constexpr int KS = (D + 15) / 16;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[2 * kStBytes];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = a.Lp >> 5, bpr = (nt + 3) >> 2;               // key tiles, blocks per (row, head)
    const int rh = blockIdx.x / bpr, jt = (blockIdx.x - rh * bpr) * 4 + wave;
    const int r = rh / a.H, h = rh - r * a.H, j0 = jt * 32, j = j0 + col;
    const bool active = jt < nt;                                 // (a block's last wavefronts may have no key tile)
    const size_t base = (size_t)rh * a.L * D;
    TileSrc src;
    src.x = a.q + base; src.y = a.dctx + base;
    src.va = a.lse + (size_t)rh * 2 * a.Lp; src.vb = a.delta + (size_t)rh * 2 * a.Lp;
    src.L = a.L; src.Lp = a.Lp;

    Frag kf[KS], vf[KS];
    load_rows<D, FULL>(kf, a.k + base, active ? j0 : 0, a.L, col, hf);
    load_rows<D, FULL>(vf, a.v + base, active ? j0 : 0, a.L, col, hf);
    const bool key_ok = active && (FULL || j < a.L) && a.mrow[(size_t)r * a.mstride + ((FULL || j < a.L) ? j : 0)] != 0.f;
    if (!key_ok)                              // (zeros, as everywhere: the content of a masked key reaches nothing)
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[s].u = vf[s].u = make_uint4(0, 0, 0, 0);
    // What the accumulator of the logits starts from (see bias_tile_fetch), here with lane = key and register v =
    // query i0 + 8(v/4) + 4hf + v%4: the bias tile times sqrt(d), and -inf in every register if the lane's key is
    // masked or beyond L.  Two sets of bias tiles (even and odd query tiles), requested ahead like the staged tiles.
    const Frag kx = key_side(key_ok, hf), one = one_side(hf);
    const int jta = active ? jt : 0;
    float4 brow[2][4];
    uint4 rs[2][2];
    StagePlan<D, FULL> plan;
    plan.init(src, tid);
    plan.fetch(0, a.L, rs[0][0], rs[0][1]);
    if (BIAS) bias_tile_fetch(brow[0], a.biasK, h, nt, 0, jta, lane);
    plan.store(s_stage, 0, a.L, rs[0][0], rs[0][1]);
    __syncthreads();

    f32x16 dk = zero16(), dv = zero16();     // dk^T, dv^T: lane = key, register = channel
#define FF_BWD_DKV_TILE(P)                                                                                       \
    {                                                                                                            \
        const int i0 = 32 * (tt + (P));                                                                          \
        const unsigned char* stage = s_stage + (P) * kStBytes;                                                   \
        constexpr int PF = 1 - (P);                                                                              \
        const int in = i0 + 32 < a.L ? i0 + 32 : i0;              /* (the last tile asks for itself again) */    \
        plan.fetch(in, a.L, rs[PF][0], rs[PF][1]);                                                               \
        f32x16 s;                                                                                                \
        if (BIAS) {                                                                                              \
            rows_to_acc(s, brow[P]);                                                                             \
            bias_tile_fetch(brow[PF], a.biasK, h, nt, in >> 5, jta, lane);                                       \
        } else {                                                                                                 \
            s = zero16();                                                                                        \
        }                                                                                                        \
        if (active) {                                                                                            \
            Frag qf[KS], dcf[KS], qt[2], dct[2], pf[2], dsf[2];                                                  \
            staged_rows<D>(qf, stage + kStRowsX, col, hf);                                                       \
            staged_rows<D>(dcf, stage + kStRowsY, col, hf);                                                      \
            f32x16 dp;        /* lane = key, register v = query i0 + 8(v/4) + 4hf + v%4; starts from -delta */   \
            _Pragma("unroll") for (int gq = 0; gq < 4; ++gq) {                                                   \
                const float4 d4 = *reinterpret_cast<const float4*>(stage + kStVecB + (8 * gq + 4 * hf) * 4);     \
                dp[4 * gq] = -d4.x; dp[4 * gq + 1] = -d4.y; dp[4 * gq + 2] = -d4.z; dp[4 * gq + 3] = -d4.w;      \
            }                                                                                                    \
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(one.v, kx.v, s, 0, 0, 0);      /* -inf for a masked key */ \
            _Pragma("unroll") for (int t = 0; t < KS; ++t) {                                                     \
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t].v, kf[t].v, s, 0, 0, 0);                       \
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dcf[t].v, vf[t].v, dp, 0, 0, 0);                    \
            }                                                                                                    \
            staged_cols(qt, stage + kStRowsX, lane);                                                             \
            staged_cols(dct, stage + kStRowsY, lane);                                                            \
            _Pragma("unroll") for (int gq = 0; gq < 4; ++gq) {                                                   \
                const float4 l4 = *reinterpret_cast<const float4*>(stage + kStVecA + (8 * gq + 4 * hf) * 4);     \
                const float ls[4] = {l4.x, l4.y, l4.z, l4.w};                                                    \
                _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                  \
                    const int v = 4 * gq + e;                                                                    \
                    /* (a query beyond L or without keys has logsumexp +inf, a masked key a logit of -inf:        \
                       weight 0 either way) */                                                                   \
                    const float p = __builtin_amdgcn_exp2f(s[v] * a.qscale2 - ls[e]);                            \
                    s[v] = p;                                                                                    \
                    dp[v] = p * dp[v];                                                                           \
                }                                                                                                \
            }                                                                                                    \
            pack_rows(pf, s);                                                                                    \
            pack_rows(dsf, dp);                                                                                  \
            _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                                      \
                dv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dct[t].v, pf[t].v, dv, 0, 0, 0);                    \
                dk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt[t].v, dsf[t].v, dk, 0, 0, 0);                    \
            }                                                                                                    \
        }                                                                                                        \
        if (i0 + 32 < a.L)                                                                                       \
            plan.store(s_stage + (1 - (P)) * kStBytes, i0 + 32, a.L, rs[1 - (P)][0], rs[1 - (P)][1]); \
        __syncthreads();                                                                                         \
    }
    for (int tt = 0; 32 * tt < a.L; tt += 2) {
        FF_BWD_DKV_TILE(0)
        if (32 * (tt + 1) < a.L) FF_BWD_DKV_TILE(1)
    }
#undef FF_BWD_DKV_TILE
    if (active && (FULL || j < a.L)) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const int e0 = 8 * gq + 4 * hf;
            if (e0 < D) {
                const size_t off = base + (size_t)j * D + e0;
                *reinterpret_cast<uint2*>(a.dv + off) = make_uint2(pack2(dv[4 * gq], dv[4 * gq + 1]), pack2(dv[4 * gq + 2], dv[4 * gq + 3]));
                *reinterpret_cast<uint2*>(a.dk + off) = make_uint2(pack2(dk[4 * gq] * a.scale, dk[4 * gq + 1] * a.scale),
                                                                   pack2(dk[4 * gq + 2] * a.scale, dk[4 * gq + 3] * a.scale));
            }
        }
    }
}

// ====================================================================================
// Up to 512 positions: statistics, dq, dk and dv of one (row, head) in one block, so that every tensor passes memory once and the
// weights are recomputed once for dq, dk and dv together.  q, k, v and later dctx of the (row, head) stay in LDS.  There is a wavefront per
// 32 positions: wavefront w owns query tile w while the statistics are formed (as k_bwd_stats), then key tile w (as
// k_bwd_dkv) and dq of query tile w.  In step s of the second phase wavefront w works on query tile (w + s) mod nt: its
// tile of dS goes to LDS (in the place of v, which is in registers by then), and after a barrier the owner of that query tile contracts it with
// the key rows of the wavefront it comes from.  The wavefronts work on different query tiles, so every one of
// them has exactly one such contraction per step.
// What bounds it: the instructions that the wavefronts of a SIMD can issue (about 130 per tile for the statistics, 190 in the second phase),
// at four wavefronts per SIMD, hence at most 128 registers (d = 16 with a bias and d = 32 without keep 28 and 12 bytes a lane in scratch memory); then the bytes.
// From nine wavefronts on a block is alone on its compute unit: 2.25 wavefronts per SIMD at 288 positions (128 rows x 8 heads x 32 with a bias 160 us the
// call, the three kernels 222; 320 181 / 247, 384 231 / 310, 448 274 / 382).  Two tiles per wavefront and two wavefronts per SIMD need fewer
// LDS reads, but took 96 us at 128 rows x 8 heads x 256 x 32 with a bias; now 77, the three kernels 117 (46 + 32 + 40).  Without its tile
// loops it takes 39 us there for the 168 MB that it moves.
// Rows are 64 bytes whatever the head dim, the 16-byte piece p of row n at p ^ (n / 4) % 4: operand reads of rows and transposing reads alike
// then spread over the banks.  Masked keys and positions beyond L are zeros; their dk and dv are not taken from the
// accumulators, and their weights are cleared from dS.
constexpr int kRowsTiles = 16;                         // at most: 32 positions per wavefront
__device__ __forceinline__ int piece_swizzle(int n) { return (n >> 2) & 3; }

// operand fragments of a swizzled tile: rows of the lane's position, lane_off = rows_lane(col, hf) ...
__device__ __forceinline__ int rows_lane(int col, int hf) { return col * 64 + ((hf ^ piece_swizzle(col)) << 4); }
template <int D>
__device__ __forceinline__ void rows_frag(Frag (&f)[(D + 15) / 16], const unsigned char* tile, int lane_off, int hf) {
#pragma unroll
    for (int s = 0; s < (D + 15) / 16; ++s) f[s].u = *reinterpret_cast<const uint4*>(tile + (lane_off ^ (32 * s)));
    if (D == 8 && hf) f[0].u = make_uint4(0, 0, 0, 0);
}
// ... and channels of the lane over the positions 16 s + 4 hf + (u < 4 ? u : u + 4) (see staged_cols), lane_off = cols_lane(lane)
__device__ __forceinline__ int cols_lane(int lane) {
    const int hf = lane >> 5, chunk = ((lane & 16) >> 2) + (lane & 3);
    return (4 * hf + ((lane >> 2) & 3)) * 64 + (((chunk >> 1) ^ hf) << 4) + (chunk & 1) * 8;
}
__device__ __forceinline__ uint2 read_tr(const unsigned char* p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)p));
}
__device__ __forceinline__ void cols_frag(Frag (&f)[2], const unsigned char* tile, int lane_off) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint2 lo = read_tr(tile + lane_off + 1024 * s), hi = read_tr(tile + (lane_off ^ 32) + 1024 * s + 512);
        f[s].u = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
}
// A transposed result tile (lane = position, register v = channel 8 (v / 4) + 4 hf + v % 4) as 16-byte pieces: words lo, hi of channel groups
// g and g + 1 (channels 4 hf .. + 1 and + 2 .. + 3) become the eight channels of group g + hf.
__device__ __forceinline__ uint4 merge_groups(uint32_t lo0, uint32_t hi0, uint32_t lo1, uint32_t hi1) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo0, lo1, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi0, hi1, false, false);
    return make_uint4(l[0], h[0], l[1], h[1]);
}
// x [D] of the lane's position, packed words w[2 g], w[2 g + 1] of channel group g
template <int D>
__device__ __forceinline__ void store_position(bf16_t* x, const uint32_t* w, int hf) {
    if constexpr (D == 8) {
        *reinterpret_cast<uint2*>(x + 4 * hf) = make_uint2(w[0], w[1]);
    } else {
#pragma unroll
        for (int g = 0; g < D / 8; g += 2)
            *reinterpret_cast<uint4*>(x + 8 * (g + hf)) = make_uint4(w[2 * g], w[2 * g + 1], w[2 * g + 2], w[2 * g + 3]);
    }
}
// the words of store_position from an accumulator (all lanes take part)
template <int D>
__device__ __forceinline__ void pack_position(uint32_t (&w)[8], const f32x16& a, float scale) {
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
        w[2 * g] = pack2(a[4 * g] * scale, a[4 * g + 1] * scale);
        w[2 * g + 1] = pack2(a[4 * g + 2] * scale, a[4 * g + 3] * scale);
    }
    if constexpr (D > 8)
#pragma unroll
        for (int g = 0; g < D / 8; g += 2) {
            const uint4 u = merge_groups(w[2 * g], w[2 * g + 1], w[2 * g + 2], w[2 * g + 3]);
            w[2 * g] = u.x; w[2 * g + 1] = u.y; w[2 * g + 2] = u.z; w[2 * g + 3] = u.w;
        }
}

__device__ __forceinline__ uint4 only_if(bool c, uint4 v) {
    const uint32_t m = c ? 0xffffffffu : 0u;
    return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
}
// products of two pairs of bf16 values, rounded to bf16
__device__ __forceinline__ uint32_t mul_pairs(uint32_t a, uint32_t b) { return pack2(lo_f32(a) * lo_f32(b), hi_f32(a) * hi_f32(b)); }

template <int D, bool BIAS>
__global__ __launch_bounds__(64 * kRowsTiles, 4) void k_bwd_rows(Args a) {
    constexpr int KS = (D + 15) / 16, PR = D / 8, NG = D / 8;      // contraction steps, 16-byte pieces of a row, channel groups
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = a.Lp >> 5;
    const int rh = blockIdx.x, r = rh / a.H, h = rh - r * a.H;
    const size_t base = (size_t)rh * a.L * D;
    unsigned char *s_q = smem, *s_k = smem + nt * 2048, *s_v = smem + nt * 4096, *s_d = smem + nt * 6144;
    float *s_lse = reinterpret_cast<float*>(smem + nt * 8192), *s_nd = s_lse + 32 * nt;       // logsumexp and -delta of the queries
    const int n = 32 * wave + col, nc = n < a.L ? n : a.L - 1;     // the lane's query, later its key
    // (without a mask a stand-in is read and not looked at: a load under a condition is a branch and a wait of its own)
    const bool has_mask = a.mask != nullptr;
    const float* mrow = has_mask ? a.mask + (size_t)r * a.L : reinterpret_cast<const float*>(a.q + base);

    // ---- q, k, v and dctx = dout * g (rounded to bf16) into LDS, everything in flight at once (a wavefront copies its own 32 positions)
    {
        constexpr int NL = (32 * PR + 63) / 64;                    // pieces per lane
        uint4 tq[NL], tk[NL], tv[NL], td[NL], tg[NL];
        float mk[NL];
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const int id = (lane + 64 * x) % (32 * PR), row = 32 * wave + id / PR, rc = row < a.L ? row : a.L - 1;
            const size_t at = base + (size_t)rc * D + 8 * (id % PR);
            tq[x] = *reinterpret_cast<const uint4*>(a.q + at);
            tk[x] = *reinterpret_cast<const uint4*>(a.k + at);
            tv[x] = *reinterpret_cast<const uint4*>(a.v + at);
            td[x] = *reinterpret_cast<const uint4*>(a.dout + at);
            tg[x] = *reinterpret_cast<const uint4*>(a.g + at);
            mk[x] = mrow[rc];
        }
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const int id = (lane + 64 * x) % (32 * PR), row = 32 * wave + id / PR;
            const bool in = row < a.L, key = in && (!has_mask || mk[x] != 0.f);
            const int at = row * 64 + (((id % PR) ^ piece_swizzle(row)) << 4);
            *reinterpret_cast<uint4*>(s_q + at) = only_if(in, tq[x]);
            *reinterpret_cast<uint4*>(s_k + at) = only_if(key, tk[x]);
            *reinterpret_cast<uint4*>(s_v + at) = only_if(key, tv[x]);
            const uint4 dc = make_uint4(mul_pairs(td[x].x, tg[x].x), mul_pairs(td[x].y, tg[x].y), mul_pairs(td[x].z, tg[x].z), mul_pairs(td[x].w, tg[x].w));
            *reinterpret_cast<uint4*>(s_d + at) = only_if(in, dc);
            if (BIAS && in) *reinterpret_cast<uint4*>(a.dctx + base + (size_t)row * D + 8 * (id % PR)) = dc;
        }
    }
    const uint32_t keep = n < a.L && (!has_mask || mrow[nc] != 0.f) ? 0xffffffffu : 0u;      // all ones if the lane's key is attended to
    // (which keys are attended to, one bit per key: in the place of the statistics, which come later)
    uint32_t* s_live = reinterpret_cast<uint32_t*>(s_lse);
    {
        const uint32_t bits = (uint32_t)__ballot(keep != 0u);
        if (lane == 0) s_live[wave] = bits;
    }
    const int row_off = rows_lane(col, hf), col_off = cols_lane(lane);
    f32x16 b = zero16();
    auto fetch_bias = [&](const float* tiles, int it, int jt) __attribute__((always_inline)) {
        float4 rows[4];
        bias_tile_fetch(rows, tiles, h, nt, it, jt, lane);
        rows_to_acc(b, rows);
    };
    if (BIAS) fetch_bias(a.biasA, wave, 0);
    __syncthreads();

    // ---- statistics (see k_bwd_stats)
    float lse, delta;
    {
        Frag qf[KS];
        rows_frag<D>(qf, s_q + wave * 2048, row_off, hf);
        const Frag one = one_side(hf);
        constexpr float kSlack = 8.f;
        float m = -1e30f, l = 0.f;
        f32x16 ctx = zero16();
        for (int jt = 0; jt < nt; ++jt) {
            Frag kf[KS], vt[2], pf[2];
            rows_frag<D>(kf, s_k + jt * 2048, row_off, hf);
            const Frag kx = key_side((s_live[jt] >> col) & 1u, hf);
            f32x16 s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx.v, one.v, b, 0, 0, 0);
            if (BIAS) fetch_bias(a.biasA, wave, jt + 1 < nt ? jt + 1 : jt);
#pragma unroll
            for (int t = 0; t < KS; ++t) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t].v, qf[t].v, s, 0, 0, 0);
            cols_frag(vt, s_v + jt * 2048, col_off);
            float tmax = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
            tmax *= a.qscale2;
            if (__builtin_amdgcn_ballot_w64(tmax > m + kSlack) != 0) {
                const float m_new = fmaxf(m, half_max(tmax));
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
                for (int v = 0; v < 16; ++v) ctx[v] *= alpha;
                l *= alpha;
                m = m_new;
            }
            float lt = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = __builtin_amdgcn_exp2f(s[v] * a.qscale2 - m);
                lt += s[v];
            }
            l += lt;
            pack_rows(pf, s);
#pragma unroll
            for (int t = 0; t < 2; ++t) ctx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vt[t].v, pf[t].v, ctx, 0, 0, 0);
        }
        // dout of the lane's query once more (it was read a moment ago)
        uint2 dov[NG], dcv[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            dov[g] = *reinterpret_cast<const uint2*>(a.dout + base + (size_t)nc * D + 8 * g + 4 * hf);
            dcv[g] = *reinterpret_cast<const uint2*>(s_d + n * 64 + ((g ^ piece_swizzle(n)) << 4) + 8 * hf);
        }
        // (all lanes take part in what follows: the two lanes of a query exchange halves; only queries below L are stored)
        const float l_tot = half_sum(l), inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        // a query without unmasked keys: logsumexp = +inf makes every recomputed weight exp2(s - inf) = 0
        lse = l_tot > 0.f && n < a.L ? m + __builtin_amdgcn_logf(l_tot) : INFINITY;
        float dl = 0.f;          // delta uses the very dctx values the other contractions read
        uint32_t wg[8];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float d_o[4] = {lo_f32(dov[g].x), hi_f32(dov[g].x), lo_f32(dov[g].y), hi_f32(dov[g].y)};
            const float dc[4] = {lo_f32(dcv[g].x), hi_f32(dcv[g].x), lo_f32(dcv[g].y), hi_f32(dcv[g].y)};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = ctx[4 * g + e] * inv;
                dl += dc[e] * c;
                ctx[4 * g + e] = d_o[e] * c;
            }
        }
        delta = half_sum(dl);
        pack_position<D>(wg, ctx, 1.f);
        if (n < a.L) store_position<D>(a.dg + base + (size_t)n * D, wg, hf);
        if (BIAS && hf == 0) {
            a.lse[(size_t)rh * 2 * a.Lp + n] = lse;
            a.delta[(size_t)rh * 2 * a.Lp + n] = delta;
        }
    }
    // ---- dq, dk, dv
    Frag vf[KS];
    rows_frag<D>(vf, s_v + wave * 2048, row_off, hf);
    if (BIAS) fetch_bias(a.biasK, wave, wave);
    __syncthreads();                 // (the key masks and v have been read)
    if (hf == 0) {
        s_lse[n] = lse;
        s_nd[n] = -delta;
    }
    __syncthreads();
    f32x16 dk = zero16(), dv = zero16(), dq = zero16();
    unsigned char* s_ds = s_v;       // [wavefront][32 keys][32 queries]
    const int row_lane = row_off, col_lane = col_off;
    int it = wave, from = wave;      // (wave + step) mod nt, (wave - step) mod nt
    for (int step = 0; step < nt; ++step) {
        // (opaque: else every LDS address of the loop is worked out before it, and some of them wait in scratch memory)
        int row_off = row_lane, col_off = col_lane;
        asm volatile("" : "+v"(row_off), "+v"(col_off));
        Frag dsf[2];
        {
            Frag qr[KS], dr[KS], kf[KS], pf[2], ft[2];
            rows_frag<D>(qr, s_q + it * 2048, row_off, hf);
            rows_frag<D>(kf, s_k + wave * 2048, row_off, hf);
#pragma unroll
            for (int c = 0; c < KS; ++c) b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qr[c].v, kf[c].v, b, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);       // (else the operands of both contractions are in registers together, and others in scratch memory)
            f32x16 dp;               // lane = key, register v = query 8 (v / 4) + 4 hf + v % 4; starts from -delta
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 d4 = *reinterpret_cast<const float4*>(s_nd + 32 * it + 8 * g + 4 * hf);
                dp[4 * g] = d4.x; dp[4 * g + 1] = d4.y; dp[4 * g + 2] = d4.z; dp[4 * g + 3] = d4.w;
            }
            rows_frag<D>(dr, s_d + it * 2048, row_off, hf);
#pragma unroll
            for (int c = 0; c < KS; ++c) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dr[c].v, vf[c].v, dp, 0, 0, 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 l4 = *reinterpret_cast<const float4*>(s_lse + 32 * it + 8 * g + 4 * hf);
                const float ls[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    b[4 * g + e] = __builtin_amdgcn_exp2f(b[4 * g + e] * a.qscale2 - ls[e]);
                    dp[4 * g + e] *= b[4 * g + e];
                }
            }
            pack_rows(pf, b);
            pack_rows(dsf, dp);
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) dsf[c].w[i] &= keep;
            const int itn = it + 1 < nt ? it + 1 : 0;
            if (BIAS) fetch_bias(a.biasK, itn, wave);
            else b = zero16();
            cols_frag(ft, s_d + it * 2048, col_off);
#pragma unroll
            for (int c = 0; c < 2; ++c) dv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[c].v, pf[c].v, dv, 0, 0, 0);
            cols_frag(ft, s_q + it * 2048, col_off);
#pragma unroll
            for (int c = 0; c < 2; ++c) dk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[c].v, dsf[c].v, dk, 0, 0, 0);
            it = itn;
        }
        __syncthreads();             // (the dS tiles of the previous step have been read)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                *reinterpret_cast<uint2*>(s_ds + wave * 2048 + col * 64 + (((2 * c + u) ^ piece_swizzle(col)) << 4) + 8 * hf) =
                    make_uint2(dsf[c].w[2 * u], dsf[c].w[2 * u + 1]);
        __syncthreads();
        // dS of the wavefront's own query tile comes from wavefront (wave - step) mod nt this time
        Frag ds[2], kc[2];
        cols_frag(ds, s_ds + from * 2048, col_off);
        cols_frag(kc, s_k + from * 2048, col_off);
#pragma unroll
        for (int c = 0; c < 2; ++c) dq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kc[c].v, ds[c].v, dq, 0, 0, 0);
        from = from > 0 ? from - 1 : nt - 1;
    }
    uint32_t wq[8], wk[8], wv[8];
    pack_position<D>(wq, dq, a.scale);
    pack_position<D>(wk, dk, a.scale);
    pack_position<D>(wv, dv, 1.f);
#pragma unroll
    for (int i = 0; i < 2 * NG; ++i) {
        wk[i] &= keep;
        wv[i] &= keep;
    }
    if (n < a.L) {
        store_position<D>(a.dq + base + (size_t)n * D, wq, hf);
        store_position<D>(a.dk + base + (size_t)n * D, wk, hf);
        store_position<D>(a.dv + base + (size_t)n * D, wv, hf);
    }
}

// ====================================================================================
// dbias: block = sixteen wavefronts = a patch of 4 x 4 tiles of one head and one chunk of batch rows; wavefront (wi, wj) sums dS of
// tile (it0 + wi, jt0 + wj) over the rows of the chunk in registers.  Per batch row the patch needs the q and dctx rows of
// four query tiles, the k and v rows of four key tiles and logsumexp and delta of its 128 queries: 33 KiB for 16 tiles, by
// loads that write LDS directly (rows swizzled by the source address) into a ring of kDbRing rows, kDbRing - 1 rows ahead, one
// barrier per row.  Positions beyond L are the last one again: their entries are not stored.
// At 128 rows x 8 heads x 256 x 32 it takes 27 us (two tiles per wavefront, two wavefronts per SIMD: 31): about 1.05 us per batch row and block,
// 85 vector instructions per tile at four wavefronts per SIMD, and at the same time 33 KiB per block and row out of L2.
constexpr int kDbRing = 4;
constexpr int kDbStage = 16 * 2048 + 1024;                // 16 operand tiles [32][64 bytes], then logsumexp [128] and delta [128]
typedef void __attribute__((address_space(3)))* lds_void;

// byte offset of an operand fragment in a staged tile of rows of 2 D bytes (its second step: ^ 32)
template <int D>
__device__ __forceinline__ int db_rows_lane(int col, int hf) {
    if (D == 32) return rows_lane(col, hf);
    return D == 16 ? col * 32 + ((hf ^ ((col >> 3) & 1)) << 4) : col * 16;
}
template <int D>
__global__ __launch_bounds__(1024, 4) void k_bwd_dbias(Args a) {
    constexpr int KS = (D + 15) / 16, TILE = 64 * D, STAGE = 16 * TILE + 1024;
    constexpr int NLW = D / 16;                            // loads of 1 KiB per wavefront and batch row; D = 8: one by each of the first eight wavefronts
    constexpr int NL = D == 8 ? 1 : NLW;
    static_assert(STAGE <= kDbStage, "a batch row fits its place in the ring");
    extern __shared__ __attribute__((aligned(16))) unsigned char s_db[];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wi = wave >> 2, wj = wave & 3;
    const int nt = a.Lp >> 5, np = (nt + 3) >> 2;
    // (an XCD takes a contiguous range of the order chunk, head, patch: the patches of a head that share operand rows share its L2)
    const int per_xcd = (int)(gridDim.x >> 3), item = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.row_chunks * a.H * np * np) return;      // (whole block)
    const int chunk = item / (a.H * np * np), rem = item - chunk * a.H * np * np;
    const int h = rem / (np * np), pp = rem - h * np * np, it0 = 4 * (pp / np), jt0 = 4 * (pp - (pp / np) * np);
    const int it = it0 + wi, jt = jt0 + wj;
    const bool active = it < nt && jt < nt;
    const int r_begin = chunk * a.rows_per_chunk;
    const int r_end = r_begin + a.rows_per_chunk < a.R ? r_begin + a.rows_per_chunk : a.R;
    if (r_begin >= r_end) return;                          // (whole block)

    // ---- the wavefront's loads: lane i of a load fills 16-byte slot i of its KiB of the stage
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lds_void)s_db);
    const char* ld_src[NL];                                // (scalar) tensor at this head of the next batch row to request
    uint32_t ld_lane[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int c = D == 8 ? wave & 7 : 16 * i + wave;                  // KiB of the stage: half a tile, a tile or two tiles
        const int o = D == 32 ? c >> 1 : (D == 16 ? c : 2 * c);
        const bf16_t* t = o < 4 ? a.q : (o < 8 ? a.dctx : (o < 12 ? a.k : a.v));
        ld_src[i] = reinterpret_cast<const char*>(t + ((size_t)r_begin * a.H + h) * a.L * D);
        const int row = D == 32 ? 16 * (c & 1) + (lane >> 2) : (D == 16 ? lane >> 1 : lane & 31);
        const int piece = D == 32 ? (lane & 3) ^ ((lane >> 4) & 3) : (D == 16 ? (lane & 1) ^ ((lane >> 4) & 1) : 0);
        const int tile = (o & 3) + (D == 8 ? lane >> 5 : 0) + (o < 8 ? it0 : jt0);
        const int pos = 32 * tile + row < a.L ? 32 * tile + row : a.L - 1;
        ld_lane[i] = (uint32_t)(pos * 2 * D + piece * 16);
    }
    // (logsumexp by lanes 0 .. 31, delta by lanes 32 .. 63, in the last wavefront)
    const int vq = 32 * it0 + 4 * col < a.Lp ? 32 * it0 + 4 * col : a.Lp - 4;
    const char* vec_src = reinterpret_cast<const char*>(a.lse + ((size_t)r_begin * a.H + h) * 2 * a.Lp);
    const uint32_t vec_lane = (uint32_t)((hf * a.Lp + vq) * 4);
    const size_t row_bytes = (size_t)a.H * a.L * D * 2, vec_row_bytes = (size_t)a.H * 2 * a.Lp * 4;
    // Requests the next batch row (past the end: the last one again, into a slot that nobody reads).  Everything moves on by additions: a CU has
    // one scalar unit for its sixteen wavefronts, and products of row numbers and strides took it half of a row's time.
    unsigned to_slot = 0;                                  // offset of the ring slot that is filled next
    int to_row = r_begin;
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (D > 8 || wave < 8) load16_to_lds(ld_src[i], ld_lane[i], lds0 + to_slot + (16 * i + wave) * 1024);
        if (wave == 15) load16_to_lds(vec_src, vec_lane, lds0 + to_slot + 16 * TILE);
        to_slot = to_slot + STAGE < kDbRing * STAGE ? to_slot + STAGE : 0;
        if (++to_row < r_end) {
#pragma unroll
            for (int i = 0; i < NL; ++i) ld_src[i] += row_bytes;
            vec_src += vec_row_bytes;
        }
    };
    f32x16 bt, acc = zero16();      // bias tile times sqrt(d), the same for every batch row; lane = query i, register v = key 8 (v / 4) + 4 hf + v % 4
    {
        float4 rows[4];
        bias_tile_fetch(rows, a.biasA, h, nt, it < nt ? it : nt - 1, jt < nt ? jt : nt - 1, lane);
        rows_to_acc(bt, rows);
    }
    // (through the scalar cache: a vector load would count among the loads of stage())
    typedef const uint32_t __attribute__((address_space(4)))* scalar_words;
    scalar_words live = (scalar_words)(uintptr_t)(a.live + (size_t)r_begin * nt + (jt < nt ? jt : nt - 1));
    uint32_t lv = *live;
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0): from here on the counter counts the loads of stage() alone
#pragma unroll
    for (int x = 0; x < kDbRing - 1; ++x) stage();
    const Frag one = one_side(hf);
    const int off = db_rows_lane<D>(col, hf);
    // the wavefront's operands of one batch row, read from LDS while the previous row's weights are formed
    Frag qf[KS], dcf[KS], kf[KS], vf[KS];
    float lse, delta;
    const unsigned char* st = s_db;                       // slot of the next row to read
    auto read = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < KS; ++c) {
            qf[c].u = *reinterpret_cast<const uint4*>(st + wi * TILE + (off ^ (32 * c)));
            kf[c].u = *reinterpret_cast<const uint4*>(st + (8 + wj) * TILE + (off ^ (32 * c)));
            dcf[c].u = *reinterpret_cast<const uint4*>(st + (4 + wi) * TILE + (off ^ (32 * c)));
            vf[c].u = *reinterpret_cast<const uint4*>(st + (12 + wj) * TILE + (off ^ (32 * c)));
        }
        if (D == 8 && hf) qf[0].u = kf[0].u = dcf[0].u = vf[0].u = make_uint4(0, 0, 0, 0);
        lse = *reinterpret_cast<const float*>(st + 16 * TILE + (wi * 32 + col) * 4);
        delta = *reinterpret_cast<const float*>(st + 16 * TILE + 512 + (wi * 32 + col) * 4);
        st = st + STAGE < s_db + kDbRing * STAGE ? st + STAGE : s_db;
    };
    // Row r has arrived when at most the loads of the AHEAD rows behind it are on their way.  (And lgkmcnt(0): the wavefront's reads of the
    // row before, whose slot is filled next, are complete.)
    constexpr int AHEAD = kDbRing - 2;
    auto arrived = [&]() __attribute__((always_inline)) {
        if (wave == 15) __builtin_amdgcn_s_waitcnt(0x0070 | AHEAD * (NLW + 1));
        else __builtin_amdgcn_s_waitcnt(0x0070 | AHEAD * NL);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    arrived();
    stage();
    if (active) read();
    for (int r = r_begin; r < r_end; ++r) {
        arrived();                                         // row r + 1; row r has been read by everybody
        stage();
        if (active) {
            const Frag kx = key_side((lv >> col) & 1u, hf);
            if (lv != 0xffffffffu) {                           // (wave-uniform: masked keys are zeros here too)
                const bool ok = (lv >> col) & 1u;
#pragma unroll
                for (int c = 0; c < KS; ++c) {
                    kf[c].u = only_if(ok, kf[c].u);
                    vf[c].u = only_if(ok, vf[c].u);
                }
            }
            f32x16 s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kx.v, one.v, bt, 0, 0, 0), dp = zero16();
#pragma unroll
            for (int c = 0; c < KS; ++c) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c].v, qf[c].v, s, 0, 0, 0);
#pragma unroll
            for (int c = 0; c < KS; ++c) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c].v, dcf[c].v, dp, 0, 0, 0);
            const float l0 = lse, d0 = delta;
            read();                                        // (past the end: a slot that holds the last row again)
            if (r + 1 < r_end) live += nt;
            lv = *live;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += __builtin_amdgcn_exp2f(s[v] * a.qscale2 - l0) * (dp[v] - d0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // (no load may write LDS after the block has ended)
    if (!active) return;
    if (a.row_chunks > 1) {
        float* part = a.dbias_part + ((((size_t)chunk * a.H + h) * nt + it) * nt + jt) * 1024 + lane * 4;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(part + 256 * g) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    } else {
        const int i = 32 * it + col;
        float* drow = a.dbias + ((size_t)h * a.L + i) * a.L;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int j = 32 * jt + 8 * (v >> 2) + 4 * hf + (v & 3);
            if (i < a.L && j < a.L) drow[j] = acc[v];
        }
    }
}

// dbias = sum over the row chunks of the partial sums, in chunk order (deterministic).  A block per tile: eight threads take the 32
// entries of a row, so that 128 bytes of a row are written together; entry 8 g + 4 hf .. of row i lies at lane 32 hf + i of group g.
__global__ __launch_bounds__(256) void k_bwd_dbias_reduce(Args a) {
    const int nt = a.Lp >> 5, tile = blockIdx.x, h = tile / (nt * nt), rem = tile - h * nt * nt;
    const int x = threadIdx.x >> 3, c = threadIdx.x & 7, i = 32 * (rem / nt) + x, j = 32 * (rem % nt) + 4 * c;
    const size_t n = (size_t)a.H * nt * nt * 1024;
    const float* p = a.dbias_part + (size_t)tile * 1024 + 256 * (c >> 1) + (32 * (c & 1) + x) * 4;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int k = 0; k < a.row_chunks; ++k) {
        const float4 y = *reinterpret_cast<const float4*>(p + k * n);
        t.x += y.x; t.y += y.y; t.z += y.z; t.w += y.w;
    }
    if (i >= a.L) return;
    float* d = a.dbias + ((size_t)h * a.L + i) * a.L + j;
    if ((a.L & 3) == 0) {
        if (j < a.L) *reinterpret_cast<float4*>(d) = t;
    } else {
        const float e[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j + k < a.L) d[k] = e[k];
    }
}

}  // namespace bwd

bool core_backward_supported(const ff_core_desc& d) {
    return d.dtype == FF_BF16 && (d.head_dim == 8 || d.head_dim == 16 || d.head_dim == 32);
}

// Row chunks of the bias gradient: enough (head, patch of 4 x 4 tiles, chunk) blocks for one per compute unit, at
// least 8 rows each.
static int dbias_chunks(const ff_core_desc& d) {
    const int nt = (d.length + 31) / 32, np = (nt + 3) / 4;
    const long patches = (long)d.heads * np * np;
    int chunks = (int)((256 + patches - 1) / patches);
    if (chunks > d.rows / 8) chunks = d.rows / 8;
    return chunks < 1 ? 1 : chunks;
}

// Whether k_bwd_rows takes the call, with a block per (row, head) and a wavefront per 32 positions, or the three kernels with their blocks of four
// tiles.  One block holds up to kRowsTiles tiles, and from nine on it is alone on its compute unit.  Up to there it is the better one at every size
// (4 to 1120 (row, head)s of 64 to 256 positions: 0.55 to 0.98 of the three kernels' time).  Two exceptions above:
//  - so few (row, head)s that most units have none: four wavefronts share a SIMD while others idle.  With ever longer sequences ever more
//    of them are too few: 4 (row, head)s, d = 32 without a bias, of 320 positions 22.2 us against 21.7, 384 26.5 / 24.4, 416 33.4 / 25.9, 512 41.3 / 29.9;
//    64 of 384 27.5 / 28.1, 416 35.0 / 30.7, 512 42.9 / 34.8; 96 of 512 44.7 / 44.0; with a bias 4 of 512 61 / 51, 64 72 / 64, 96 74 / 74.
//  - more than there are units by so few that the second round is nearly empty, without a bias: 264 of 512 positions at d = 8 take 75.5 us against 68.0, at
//    d = 16 77.4 / 71.3, 320 76.5 / 69.8 and 77.8 / 74.7, of 384 48.0 / 45.4 and 49.4 / 48.6; the three kernels' time steps up where their
//    blocks begin another round (336 of 512 at d = 8 76.7 / 79.4).  At d = 32 264 of 512 92.1 / 89.8, 296 92.6 / 92.7, of 384 58.9 / 59.6.  With a
//    bias the three kernels read its tiles three times: 264 of 512 at d = 16 121 / 118, else never.
static bool rows_in_lds(const ff_core_desc& d, int nt, bool bias) {
    const int64_t rh = (int64_t)d.rows * d.heads, cu = compute_units();
    if (nt > bwd::kRowsTiles) return false;
    if (nt < 9) return true;
    if (8 * rh <= cu * ((nt - 9) / 2)) return false;
    if (bias || rh <= cu) return true;
    const int fours = (nt + 3) / 4;
    return d.head_dim == 32 ? nt < 13 || 8 * rh > 9 * cu : rh * fours > (fours + 1) * cu;
}

size_t core_backward_workspace(const ff_core_desc& d) {
    const size_t Lp = bwd::round_up(d.length, 32), rh = (size_t)d.rows * d.heads;
    const int chunks = dbias_chunks(d);
    return bwd::align256(Lp * 4) + bwd::align256(2 * rh * Lp * 4) + bwd::align256((size_t)d.rows * (Lp / 32) * 4) +
           bwd::align256(rh * d.length * d.head_dim * 2) + 2 * bwd::align256((size_t)d.heads * Lp * Lp * 4) +
           (chunks > 1 ? bwd::align256((size_t)chunks * d.heads * Lp * Lp * 4) : 0);
}

ff_status core_backward_run(const ff_core_desc& d, const void* q, const void* k, const void* v, const void* g, const float* bias,
                            const float* mask, const void* dout, void* dq, void* dk, void* dv, void* dg, float* dbias,
                            void* ws, hipStream_t st) {
    using namespace bwd;
    Args a{};
    a.q = (const bf16_t*)q; a.k = (const bf16_t*)k; a.v = (const bf16_t*)v; a.g = (const bf16_t*)g; a.dout = (const bf16_t*)dout;
    a.bias = bias; a.mask = mask; a.dq = (bf16_t*)dq; a.dk = (bf16_t*)dk; a.dv = (bf16_t*)dv; a.dg = (bf16_t*)dg; a.dbias = dbias;
    a.R = d.rows; a.H = d.heads; a.L = d.length; a.Lp = round_up(d.length, 32);
    const size_t rh = (size_t)d.rows * d.heads;
    char* p = (char*)ws;
    a.ones = (float*)p; p += align256((size_t)a.Lp * 4);
    a.mrow = mask ? mask : a.ones;
    a.mstride = mask ? d.length : 0;
    a.lse = (float*)p; p += align256(2 * rh * a.Lp * 4);
    a.delta = a.lse + a.Lp;
    a.live = (uint32_t*)p; p += align256((size_t)d.rows * (a.Lp / 32) * 4);
    a.dctx = (bf16_t*)p; p += align256(rh * d.length * d.head_dim * 2);
    const size_t bbytes = align256((size_t)d.heads * a.Lp * a.Lp * 4);
    a.biasA = (float*)p; p += bbytes;
    a.biasK = (float*)p; p += bbytes;
    a.row_chunks = bias ? dbias_chunks(d) : 1;
    a.rows_per_chunk = (d.rows + a.row_chunks - 1) / a.row_chunks;
    // (rounding the share up can leave the last chunks without rows, and nobody writes their partial sums: 81 rows in
    // ten shares of 9 are nine chunks)
    a.row_chunks = (d.rows + a.rows_per_chunk - 1) / a.rows_per_chunk;
    a.dbias_part = a.row_chunks > 1 ? (float*)p : nullptr;
    a.qscale2 = kLog2e / sqrtf((float)d.head_dim);
    a.scale = 1.f / sqrtf((float)d.head_dim);
    a.sqrt_d = sqrtf((float)d.head_dim);
    const int nt = a.Lp / 32;
    const bool full = d.length % 32 == 0;        // nothing out of range: the kernels without bounds checks
#define FF_BWD_D(KERNEL, GRID, DV)                                                                       \
    do {                                                                                                 \
        if (full && bias) hipLaunchKernelGGL((KERNEL<DV, true, true>), GRID, dim3(256), 0, st, a);       \
        else if (full) hipLaunchKernelGGL((KERNEL<DV, true, false>), GRID, dim3(256), 0, st, a);         \
        else if (bias) hipLaunchKernelGGL((KERNEL<DV, false, true>), GRID, dim3(256), 0, st, a);         \
        else hipLaunchKernelGGL((KERNEL<DV, false, false>), GRID, dim3(256), 0, st, a);                  \
    } while (0)
#define FF_BWD(KERNEL, GRID, KIND)                                                                       \
    do {                                                                                                 \
        Timed t(KIND, st);                                                                               \
        if (d.head_dim == 8) FF_BWD_D(KERNEL, GRID, 8);                                                  \
        else if (d.head_dim == 16) FF_BWD_D(KERNEL, GRID, 16);                                           \
        else FF_BWD_D(KERNEL, GRID, 32);                                                                 \
    } while (0)
    const bool in_lds = rows_in_lds(d, nt, bias != nullptr);
    if (bias || (!mask && !in_lds)) {
        Timed t(KK_BWD_PREPARE, st);
        const size_t tasks = bias ? (size_t)d.heads * nt * nt + (size_t)d.rows * ((nt + 1) / 2) : 1;
        hipLaunchKernelGGL(k_bwd_prepare, dim3((unsigned)((tasks + 3) / 4)), dim3(256), 0, st, a);
    }
    hipError_t attr = hipSuccess;
    if (in_lds) {
        Timed t(KK_BWD_ROWS, st);
        constexpr int lds_tile = 4 * 2048 + 2 * 128;         // q, k, v, dctx, logsumexp and delta of 32 positions
#define FF_BWD_ROWS(DV, BV)                                                                                      \
    do {                                                                                                         \
        static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bwd_rows<DV, BV>),  \
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, kRowsTiles * lds_tile); \
        attr = once;                                                                                             \
        if (once == hipSuccess) hipLaunchKernelGGL((k_bwd_rows<DV, BV>), dim3((unsigned)rh), dim3(64 * nt), nt * lds_tile, st, a); \
    } while (0)
        if (d.head_dim == 8) { if (bias) FF_BWD_ROWS(8, true); else FF_BWD_ROWS(8, false); }
        else if (d.head_dim == 16) { if (bias) FF_BWD_ROWS(16, true); else FF_BWD_ROWS(16, false); }
        else { if (bias) FF_BWD_ROWS(32, true); else FF_BWD_ROWS(32, false); }
#undef FF_BWD_ROWS
        if (attr != hipSuccess) return fail(FF_EHIP, "k_bwd_rows: dynamic LDS limit: %s", hipGetErrorString(attr));
    } else {
        const dim3 g4((unsigned)(rh * ((nt + 3) / 4)));      // blocks of four tiles of one (row, head)
        FF_BWD(k_bwd_stats, g4, KK_BWD_STATS);
        FF_BWD(k_bwd_dq, g4, KK_BWD_DQ);
        FF_BWD(k_bwd_dkv, g4, KK_BWD_DKV);
    }
#undef FF_BWD
#undef FF_BWD_D
    if (bias) {
        {
            Timed t(KK_BWD_DBIAS, st);
            const dim3 g2((unsigned)(((size_t)a.row_chunks * d.heads * ((nt + 3) / 4) * ((nt + 3) / 4) + 7) / 8 * 8));
#define FF_BWD_DB(DV)                                                                                            \
    do {                                                                                                         \
        constexpr int lds = kDbRing * (16 * 64 * DV + 1024);                                                     \
        static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bwd_dbias<DV>),     \
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);    \
        attr = once;                                                                                             \
        if (once == hipSuccess) hipLaunchKernelGGL((k_bwd_dbias<DV>), g2, dim3(1024), lds, st, a);               \
    } while (0)
            if (d.head_dim == 8) FF_BWD_DB(8);
            else if (d.head_dim == 16) FF_BWD_DB(16);
            else FF_BWD_DB(32);
#undef FF_BWD_DB
            if (attr != hipSuccess) return fail(FF_EHIP, "k_bwd_dbias: dynamic LDS limit: %s", hipGetErrorString(attr));
        }
        if (a.row_chunks > 1) {
            Timed t(KK_BWD_DBIAS_REDUCE, st);
            hipLaunchKernelGGL(k_bwd_dbias_reduce, dim3((unsigned)((size_t)d.heads * nt * nt)), dim3(256), 0, st, a);
        }
    }
    return check_launch("attention core backward");
}

}  // namespace ff
