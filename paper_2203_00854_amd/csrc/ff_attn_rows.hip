// Attention of the bf16 matrix-core family (FastFold Section 5.2's fused scale + mask + bias softmax between the two
// contractions) at head dimensions 8, 16 and 32, for the calls that k_proj_attn does not take.
//
// A wavefront owns 32 queries of NR batch rows and walks over the keys in steps of 32: NR tiles of 32 x 32 scores
// per step, S^T = K Q^T with the pair-bias tile as accumulator input, exponentials, O^T += V^T P^T.  The bias tile
// does not depend on the batch row, so it is loaded once per step, in accumulator register order (bias_index), straight
// into the registers that the first matrix instruction of all NR rows reads.  k and v^T of the NR rows are
// the same for all NW wavefronts of a block (they hold other queries): they pass through a ring of four steps
// in LDS, filled by loads that write LDS directly, three steps ahead, with one barrier per step.
//
// The vector unit and the matrix cores bound it together: per tile 16 exponentials (8 cycles each) and 8 packs (4)
// against four 32 x 32 x 16 matrix instructions (32 each) and two 16 x 16 x 32 ones for the denominator, so nothing else is
// left in the loop:
//  - no reference is subtracted from the scores.  float32 and bfloat16 keep their relative precision over the whole
//    exponent range, so exp2(s) / sum exp2(s) needs none while the sums stay in range; a row of a
//    wavefront whose sums do not is done again with a running maximum (softmax_stands, end of the kernel).  That second pass is not
//    pipelined: with the logsumexp of one head's queries beyond [-41, 66] (a pair bias offset by 97) 333 x 333 triangle attention takes
//    190 us instead of 120, 1024 x 1024 in chunks 2910 instead of 1420 (its operands requested a tile ahead: 2720, but the
//    ordinary 333 call then takes 4 % more).
//  - the denominator is summed from the rounded weights by two 16 x 16 x 32 matrix instructions (add_piece): eight v_dot2 per tile do not overlap
//    with matrix instructions (bare loops of the tile's mix, two wavefronts per SIMD: 123 ns with dots, 104 with four 4 x 4 x 4
//    matrix instructions, 93 without any denominator); with those four instead of the two 2048 x 2048 in chunks takes 8291 us, 8200 so.
//    Below head dim 32 the context's matrix instructions have rows to spare: a row of ones in v^T sums the denominator.
//  - masked keys cost one more matrix instruction, in steps that hold any; steps before the first masked key skip the test.
//  - matrix instructions of the next and the previous tile alternate with the exponentials of this one.
// Measured, 64 rows x 4 heads x 2048^2 with bias: 249 us for the kernel before (a wavefront per batch row with 64 queries,
// bias through LDS, five matrix instructions per tile), 190 now; 333 rows x 4 x 333^2: 81 -> 58.  Without its loads the
// kernel takes 164, without the LDS reads as well 135; the shader clock is 2.0 - 2.1 GHz under this load (2.37 without).
// 384 columns x 8 heads of 8 x 1024^2: 534 -> 409 us (the exponentials and packs alone: about 250).
#include "ff_attn_rows.h"

namespace ff {

typedef void __attribute__((address_space(3)))* lptr_t;

namespace {

// steps in the LDS ring: blocks of two wavefronts take sequences of at most two steps (launch_d), which are in LDS from the start
constexpr int ring_of(int NW) { return NW == 2 ? 2 : 4; }

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

}  // namespace

// wavefronts per SIMD the registers of an instantiation are held to.  Without a bias and below head dim 32 two rows are held to 128
// registers: four wavefronts per SIMD, where the exponentials of a wavefront hide
// another's waits (1024-sequence column attention at d = 8, the whole call: 438 us; three wavefronts 456; four rows and
// three wavefronts 499, two 469).  Blocks of two wavefronts: three per SIMD fit without spills (64 x 384 columns at d = 8:
// 8.1 us, with four 10.4).
constexpr int attn_rows_waves(int D, int NW, bool has_bias) { return has_bias ? 2 : (NW == 2 ? 3 : (D == 32 ? 2 : 4)); }

template <int D, int NR, int NW, bool HAS_BIAS>
__global__ __launch_bounds__(NW * 64, attn_rows_waves(D, NW, HAS_BIAS)) void k_attn_rows(AttnRowsArgs a) {
    static_assert((D == 8 || D == 16 || D == 32) && (NR == 2 || NR == 4), "head dimension, rows per wavefront");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int kRing = ring_of(NW);
    constexpr int TILE = 64 * D;                    // bytes of a tile of 32 keys: k as [key][D], v^T as [D][key]
    constexpr int KS = D / 16 > 0 ? D / 16 : 1;     // contraction steps of S^T
    constexpr int STEP = NR * 2 * TILE;             // bytes of a ring slot; k and v^T of its row j:
    constexpr auto k_at = [](int j) { return D == 8 ? (j >> 1) * 4 * TILE + (j & 1) * TILE : j * 2 * TILE; };
    constexpr auto v_at = [](int j) { return D == 8 ? (j >> 1) * 4 * TILE + (j & 1) * TILE + 2 * TILE : j * 2 * TILE + TILE; };
    // below head dim 32 rows D .. 31 of the v^T operand are free: row D holds ones, so that the context's matrix
    // instructions sum the denominator; the lanes of rows D .. 31 read it from an area of alternating 64-byte blocks of ones and zeros
    constexpr bool ONES = D < 32;
    unsigned char* s_ones = smem + kRing * STEP;                                                   // [STEP]
    uint32_t* s_live = reinterpret_cast<uint32_t*>(smem + (kRing + (ONES ? 1 : 0)) * STEP);        // [key tile][NR]: bit = key is attended to

    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- which rows, head and queries.  Work-groups go to the 8 XCDs round-robin and every XCD has its own L2:
    // an XCD takes a contiguous range of the order (head, group of 8 row blocks, query block, row block inside the
    // group), so that the blocks it runs at about the same time share k and v^T (same rows) eight ways and the
    // bias (same queries) eight ways.
    int lg;
    {
        const int per_xcd = (a.n_items + 7) >> 3;
        const int slot = blockIdx.x >> 3;
        lg = (blockIdx.x & 7) * per_xcd + slot;
        if (slot >= per_xcd || lg >= a.n_items) return;      // (whole block)
    }
    const int h = lg / (a.n_rb * a.n_qb);
    int rem = lg - h * a.n_rb * a.n_qb;
    const int grp = rem / (8 * a.n_qb);
    rem -= grp * 8 * a.n_qb;
    const int gsz = a.n_rb - 8 * grp < 8 ? a.n_rb - 8 * grp : 8;
    const int qb = rem / gsz;
    const int rb = 8 * grp + rem - qb * gsz;
    const int nt = (a.L + 31) >> 5;                           // key tiles; also query tiles
    const int qt = qb * NW + wave;
    const bool active = qt < nt;                              // (wave-uniform)
    int row[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) row[j] = rb * NR + j < a.rows ? rb * NR + j : a.rows - 1;

    // ---- k and v^T on their way into the ring, a KiB per wavefront and load: lane i fills 16-byte slot i of the chunk, and
    // the piece it fetches is chosen so that the operand reads below spread over the banks (sixteen lanes at a time
    // read one 16-byte piece each): piece p of element e of v^T sits at slot 4 e + (p ^ (e / 4) % 4), piece p of key r at slot
    // 4 r + (p ^ (r / 4) % 4), 2 r + (p ^ (r / 8) % 2) or r for 32, 16 or 8 elements.
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)smem);
    const size_t head_elems = (size_t)a.Lp * D;
    constexpr int CHUNKS = STEP / 1024, CPW = (CHUNKS + NW - 1) / NW;      // of a step, and of them per wavefront
    const char* st_src[CPW];                                  // (scalar) the chunk in key tile 0
    uint32_t st_lane[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = i * NW + wave;
        // chunk c: D = 32: half c % 2 of k (c % 4 < 2) or v^T of row c / 4; D = 16: k or v^T of row c / 2; D = 8: k or v^T of rows c, c + 1 (c even)
        const int j = D == 32 ? c >> 2 : (D == 16 ? c >> 1 : c & ~1);
        const bool is_v = D == 32 ? (c & 2) != 0 : (c & 1) != 0;
        auto clamp_row = [&](int jj) __attribute__((always_inline)) { return rb * NR + jj < a.rows ? rb * NR + jj : a.rows - 1; };
        const int r0 = clamp_row(j);
        st_src[i] = reinterpret_cast<const char*>((is_v ? a.vt : a.k) + ((size_t)r0 * a.H + h) * head_elems + (D == 32 ? (c & 1) * 512 : 0));
        const uint32_t v_piece = (uint32_t)((lane & 3) ^ ((lane >> 4) & 3));           // (element lane / 4 of the chunk)
        uint32_t off = (uint32_t)(lane >> 2) * 64 + v_piece * 16;
        if (D == 16 && !is_v) off = (uint32_t)(lane >> 1) * 32 + (uint32_t)((lane & 1) ^ ((lane >> 4) & 1)) * 16;
        if (D == 8) {
            const int i5 = lane & 31;
            off = is_v ? (uint32_t)(i5 >> 2) * 64 + (uint32_t)((i5 & 3) ^ ((i5 >> 4) & 3)) * 16 : (uint32_t)i5 * 16;
            if (lane >= 32) off += (uint32_t)((size_t)(clamp_row(j + 1) - r0) * a.H * head_elems * 2);
        }
        st_lane[i] = off;
    }
    auto stage = [&](int kt) __attribute__((always_inline)) {
        const unsigned dst = lds0 + (unsigned)(kt & (kRing - 1)) * STEP + wave * 1024;
#pragma unroll
        for (int i = 0; i < CPW; ++i)
            if (CHUNKS % NW == 0 || i * NW + wave < CHUNKS) load16_to_lds(st_src[i], st_lane[i] + (uint32_t)kt * TILE, dst + i * NW * 1024);
    };
    // ---- mask entries of 64 keys per load, eight loads in flight (the ballots follow below)
    const int n_pairs = (nt + 1) >> 1;
    float mv[8];
    auto load_mask = [&](int i0) __attribute__((always_inline)) {
        if (a.mask == nullptr) return;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = i0 + m * NW;
            int r = rb * NR + i % NR, l = 64 * (i / NR) + lane;
            if (r > a.rows - 1) r = a.rows - 1;
            if (l > a.L - 1) l = a.L - 1;
            mv[m] = a.mask[(int64_t)(a.r0 + r) * a.sr + (int64_t)l * a.sl];
        }
    };
#pragma unroll
    for (int m = 0; m < 8; ++m) mv[m] = 1.f;
    load_mask(wave);
    stage(0);
    if (nt > 1) stage(1);
    if (kRing > 2 && nt > 2) stage(2);

    // ---- q: B operand of S^T (lane = query, 8 consecutive elements)
    Frag qf[NR][KS];
    const int qtc = active ? qt : nt - 1;
    const uint32_t q_lane = (uint32_t)(col * D + (D > 8 ? 8 * hf : 0)) * 2;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const bf16_t* qp = a.q + ((size_t)row[j] * a.H + h) * head_elems + (size_t)qtc * (32 * D);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qf[j][s].u = ldg16(qp + 16 * s, q_lane);
            if (D == 8 && hf != 0) qf[j][s].u = make_uint4(0, 0, 0, 0);      // (the upper half of the contraction is empty)
        }
    }
    // ---- bias tiles of the wavefront's queries, one after the other
    const float* bias_q = HAS_BIAS ? a.bias + ((size_t)h * (a.Lq >> 5) + qtc) * (a.Lp >> 5) * 1024 : nullptr;
    // (the lane of a query beyond L takes the last real one's: nobody has written its own, and the denominators multiply its weights by zero)
    const int last_q = a.L - 1 - 32 * qtc;
    const uint32_t b_lane = (uint32_t)((col < last_q ? col : last_q) + 32 * hf) * 16;
    auto load_bias = [&](int kt, f32x16& b, uint32_t off) __attribute__((always_inline)) {
        if constexpr (HAS_BIAS) {
            if (kt > nt - 1) kt = nt - 1;
            const char* bp = reinterpret_cast<const char*>(bias_q + (size_t)kt * 1024);
            asm volatile("" : "+v"(off));
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 x4 = *reinterpret_cast<const float4*>(bp + g * 1024 + off);
                b[4 * g] = x4.x; b[4 * g + 1] = x4.y; b[4 * g + 2] = x4.z; b[4 * g + 3] = x4.w;
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) b[v] = 0.f;
        }
    };
    f32x16 bias_a, bias_b;
    load_bias(0, bias_a, b_lane);
    load_bias(1, bias_b, b_lane);

    // ---- which keys are attended to, one bit per key
    for (int i0 = wave; i0 < NR * n_pairs; i0 += 8 * NW) {
        if (i0 != wave) load_mask(i0);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = i0 + m * NW, j = i % NR, pair = i / NR;
            const uint64_t bits = __ballot(mv[m] != 0.f && 64 * pair + lane < a.L);
            if (lane == 0 && pair < n_pairs) {
                s_live[(2 * pair) * NR + j] = (uint32_t)bits;
                s_live[(2 * pair + 1) * NR + j] = (uint32_t)(bits >> 32);
            }
        }
    }
    if constexpr (ONES) {
        for (int i = tid; i < STEP / 16; i += NW * 64) {
            const uint32_t v = i & 4 ? 0u : 0x3f803f80u;
            *reinterpret_cast<uint4*>(s_ones + i * 16) = make_uint4(v, v, v, v);
        }
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();

    // permuted key of S^T row m = col: the lane's registers 8c .. 8c+7 then hold the keys 16c + 8hf .. + 7
    const int kperm = 16 * (col >> 4) + 8 * ((col >> 2) & 1) + 4 * ((col >> 3) & 1) + (col & 3);
    const uint32_t rd_k = D == 32 ? (uint32_t)(kperm * 64 + ((hf ^ ((kperm >> 2) & 3)) * 16))
                                  : (D == 16 ? (uint32_t)(kperm * 32 + ((hf ^ ((kperm >> 3) & 1)) * 16)) : (uint32_t)(kperm * 16));
    // (rows D .. 31 of v^T do not move with the ring slot; their pieces lie in the banks that rows 0 .. 7 leave free)
    const bool v_row = col < D;
    const uint32_t rd_v = v_row ? (uint32_t)(col * 64 + ((hf ^ ((col >> 2) & 3)) * 16))
                                : (uint32_t)(kRing * STEP + (col == D ? 0 : 64) + (hf ^ 2) * 16);
    const uint32_t v_moves = v_row ? 0xffffffffu : 0u;
    auto lds16 = [&](uint32_t off) __attribute__((always_inline)) { return *reinterpret_cast<const uint4*>(smem + off); };

    // Steps before the first one that holds a masked (or missing) key have a loop of their own without the mask tests; steps behind the
    // last one that holds a valid key are left out (and the content of padding there is irrelevant).
    int n_plain = nt, n_live = 0;
    for (int i = 0; i < nt * NR; i += 64) {
        const uint32_t w = i + lane < nt * NR ? s_live[i + lane] : 0u;
        const uint64_t part = __ballot(i + lane < nt * NR && w != 0xffffffffu), some = __ballot(w != 0u);
        if (part && n_plain == nt) n_plain = (i + (int)__builtin_ctzll(part)) / NR;
        if (some) n_live = (i + 63 - (int)__builtin_clzll(some)) / NR + 1;
    }
    // publishes what set out a step ago and sends the next step on its way (the ring slot it fills was last read before
    // the barrier)
    auto turn = [&](int kt) __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (kRing > 2 && kt + 3 < n_live) stage(kt + 3);
    };
    if (!active) {                                            // (no queries: only the share of the loads)
        for (int kt = 0; kt < n_live; ++kt) turn(kt);
        return;
    }

    f32x16 o_acc[NR], s_acc[2];
    float l_run[NR];          // denominators (head dim 32; below it they are a row of o_acc)
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        l_run[j] = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) o_acc[j][v] = 0.f;
    }
    Frag kf[2][KS], vf[2][2], pf[2];
    const bf16x8 sel = sum_select(lane);
#pragma unroll
    for (int c = 0; c < 2; ++c) pf[c].u = vf[1][c].u = make_uint4(0, 0, 0, 0);
    // One tile (row j of the step) of the software pipeline: the exponentials of tile t run while the matrix core forms
    // the scores of tile t + 1 (bias bn, query operand qn, keys kn) and the context of tile t - 1 (weights pp, values vp),
    // and the operands k of tile t + 2 and v^T of tile t come from LDS.
    auto tile = [&](auto plain_c, uint32_t live, f32x16& sc, f32x16& sn, const f32x16& bn, Frag (&kn)[KS], Frag (&kl)[KS], Frag (&vp)[2], Frag (&vl)[2], Frag (&qn)[KS], uint32_t kl_off, uint32_t vl_off0, uint32_t vl_off1,
                    f32x16& op, float& lp) __attribute__((always_inline)) {
        Frag pc[2];
        f32x4 lt = {0.f, 0.f, 0.f, 0.f};
        float e0 = __builtin_amdgcn_exp2f(sc[0]), e1 = __builtin_amdgcn_exp2f(sc[1]);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if (g == 0) sn = mfma(kn[0].v, qn[0].v, bn);
            if (KS > 1 && g == 2) sn = mfma(kn[KS - 1].v, qn[KS - 1].v, sn);
            if (g == 4) op = mfma(vp[0].v, pf[0].v, op);
            if (g == 6) op = mfma(vp[1].v, pf[1].v, op);
            if (!decltype(plain_c)::value && g == 4 && live != 0xffffffffu) sn = mask_step(live, kperm, hf, sn);
            if (!ONES && (g & 3) == 3) lt = add_piece(sel, pf[g >> 2].v, lt);
            if (g == 0) {
                kl[0].u = lds16(kl_off + rd_k);
                if (KS > 1) kl[KS - 1].u = lds16(kl_off + (rd_k ^ 32u));
            }
            if (g == 1) {
                vl[0].u = lds16(ONES ? vl_off0 : vl_off0 + rd_v);
                vl[1].u = lds16(ONES ? vl_off1 : vl_off0 + (rd_v ^ 32u));
            }
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
        if (!ONES) lp += lt[0];
        pf[0] = pc[0];
        pf[1] = pc[1];
    };
    // A step: NR tiles.  bc: bias of this step, bn: of the next one (its registers receive the one after next).
    uint32_t live_c[NR], live_n[NR];           // keys of this step (scalar) and the next
    auto fetch_live = [&](int kt, uint32_t (&lv)[NR]) __attribute__((always_inline)) {
        if (kt > nt - 1) kt = nt - 1;
#pragma unroll
        for (int j = 0; j < NR; ++j) lv[j] = s_live[kt * NR + j];
    };
    auto step = [&](auto plain_c, int kt, f32x16& bc, f32x16& bn) __attribute__((always_inline)) {
        const uint32_t cur = (uint32_t)(kt & (kRing - 1)) * STEP, nxt = (uint32_t)((kt + 1) & (kRing - 1)) * STEP;
        constexpr bool PLAIN = decltype(plain_c)::value;
        if constexpr (!PLAIN) fetch_live(kt + 1, live_n);
        const uint32_t v0 = ONES ? rd_v + (cur & v_moves) : cur, v1 = ONES ? (rd_v ^ 32u) + (cur & v_moves) : cur;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            constexpr int LAST = NR - 1;
            if (j == LAST) {
                turn(kt);
                if constexpr (!PLAIN)
#pragma unroll
                for (int i = 0; i < NR; ++i) live_n[i] = __builtin_amdgcn_readfirstlane(live_n[i]);
            }
            const uint32_t kl_off = j + 2 < NR ? cur + k_at(j + 2) : nxt + k_at(j + 2 - NR);
            Frag(&qn)[KS] = qf[j == LAST ? 0 : j + 1];
            f32x16& op = o_acc[j == 0 ? LAST : j - 1];
            const f32x16& bt = j == LAST ? bn : bc;
            tile(plain_c, j == LAST ? live_n[0] : live_c[j == LAST ? 0 : j + 1], s_acc[j & 1], s_acc[(j + 1) & 1], bt, kf[(j + 1) & 1],
                 kf[j & 1], vf[(j + 1) & 1], vf[j & 1], qn, kl_off, v0 + v_at(j), v1 + v_at(j), op, l_run[j == 0 ? LAST : j - 1]);
            if (j == LAST) load_bias(kt + 2, bc, b_lane);
        }
        if constexpr (!PLAIN) {
#pragma unroll
            for (int j = 0; j < NR; ++j) live_c[j] = live_n[j];
        }
    };

    // ---- the scores of the first tile
    fetch_live(0, live_c);
#pragma unroll
    for (int j = 0; j < NR; ++j) live_c[j] = __builtin_amdgcn_readfirstlane(live_c[j]);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        kf[0][s].u = lds16(rd_k ^ (32u * s));
        s_acc[0] = mfma(kf[0][s].v, qf[0][s].v, s == 0 ? bias_a : s_acc[0]);
        kf[1][s].u = lds16(k_at(1) + (rd_k ^ (32u * s)));
    }
    s_acc[0] = mask_step(live_c[0], kperm, hf, s_acc[0]);
    int kt = 0;
    using std::integral_constant;
    for (; kt + 2 < n_plain; kt += 2) {                       // (a step also forms the first scores of the next one)
        step(integral_constant<bool, true>{}, kt, bias_a, bias_b);
        step(integral_constant<bool, true>{}, kt + 1, bias_b, bias_a);
    }
    fetch_live(kt, live_c);
#pragma unroll
    for (int j = 0; j < NR; ++j) live_c[j] = __builtin_amdgcn_readfirstlane(live_c[j]);
    for (; kt + 1 < n_live; kt += 2) {
        step(integral_constant<bool, false>{}, kt, bias_a, bias_b);
        step(integral_constant<bool, false>{}, kt + 1, bias_b, bias_a);
    }
    if (kt < n_live) step(integral_constant<bool, false>{}, kt, bias_a, bias_b);
    o_acc[NR - 1] = mfma(vf[1][0].v, pf[0].v, o_acc[NR - 1]);
    o_acc[NR - 1] = mfma(vf[1][1].v, pf[1].v, o_acc[NR - 1]);
    if constexpr (!ONES) {
        f32x4 lt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c) lt = add_piece(sel, pf[c].v, lt);
        l_run[NR - 1] += lt[0];
    }

    // ---- normalise, gate, store.  Lane = query, register v = element 8*(v/4) + 4*hf + v%4
    // (the lane's indices anew: those from the beginning of the kernel would be held in registers through the steps, of which there are none left: without
    // this three to five went to scratch memory, and a kernel that uses it starts later.  1024 x 384 columns at d = 8 430 us the call instead of 426, 60 x 300
    // row attention 61.3 instead of 59.9)
    const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), ecol = ln & 31, ehf = ln >> 5;
    const uint32_t eq_lane = (uint32_t)(ecol * D + (D > 8 ? 8 * ehf : 0)) * 2;
    const int qi = 32 * qt + ecol;
    auto load_gate = [&](int r, uint2 (&gr)[D / 8]) __attribute__((always_inline)) {
        const bf16_t* gp = a.g + ((size_t)r * a.H + h) * head_elems + (size_t)qt * (32 * D);
#pragma unroll
        for (int g = 0; g < D / 8; ++g)
            gr[g] = *reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(gp + 8 * g) + (uint32_t)(ecol * D + 4 * ehf) * 2);
    };
    auto finish = [&](const f32x16& o, float l_tot, int r, const uint2 (&gate)[D / 8]) __attribute__((always_inline)) {
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        const size_t off = ((size_t)r * a.H + h) * head_elems + (size_t)qt * (32 * D);
        uint32_t pk[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            const uint2 gr = gate[g];
            pk[2 * g] = pack2(o[4 * g] * inv * lo_f32(gr.x), o[4 * g + 1] * inv * hi_f32(gr.x));
            pk[2 * g + 1] = pack2(o[4 * g + 2] * inv * lo_f32(gr.y), o[4 * g + 3] * inv * hi_f32(gr.y));
        }
        merge_halves(pk[0], pk[2]);      // lower half-wave: e 0..7, upper: e 8..15
        merge_halves(pk[1], pk[3]);
        merge_halves(pk[4], pk[6]);      // lower: e 16..23, upper: e 24..31
        merge_halves(pk[5], pk[7]);
        if (qi < a.L && (D > 8 || ehf == 0)) {
            char* op = reinterpret_cast<char*>(a.o + off) + eq_lane;
            *reinterpret_cast<uint4*>(op) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            if (D == 32) *reinterpret_cast<uint4*>(op + 32) = make_uint4(pk[4], pk[5], pk[6], pk[7]);
        }
    };
    // the denominator of the lane's query: both halves' partial sums, or row D of the context
    auto denominator = [&](const f32x16& o, float l) __attribute__((always_inline)) {
        if constexpr (!ONES) return l;
        const float x = o[ONES ? D / 2 : 0], y = other_half(x);      // (row D: register D / 2 of the lower half-wave)
        return ehf == 0 ? x : y;
    };
    // rows that do not stand (softmax_stands) are done again below
    int again = 0;
    uint2 gate[NR][D / 8];
#pragma unroll
    for (int j = 0; j < NR; ++j) load_gate(row[j], gate[j]);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const float l_tot = denominator(o_acc[j], l_run[j]);
        if (rb * NR + j >= a.rows) continue;
        if (__any(!softmax_stands<D / 2>(o_acc[j], l_tot) && qi < a.L)) again |= 1 << j;
        else finish(o_acc[j], l_tot, row[j], gate[j]);
    }
    // ---- the general softmax, one row after the other, operands straight from memory
    while (again != 0) {
        const int j = __builtin_ctz(again);
        again &= again - 1;
        const int r = rb * NR + j;
        const size_t off = ((size_t)r * a.H + h) * head_elems;
        Frag qs[KS];
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            qs[i].u = ldg16(a.q + off + (size_t)qt * (32 * D) + 16 * i, eq_lane);
            if (D == 8 && ehf != 0) qs[i].u = make_uint4(0, 0, 0, 0);
        }
        f32x16 o;
#pragma unroll
        for (int v = 0; v < 16; ++v) o[v] = 0.f;
        float m = -INFINITY, l = 0.f;
        for (int kt = 0; kt < nt; ++kt) {
            const uint32_t live = __builtin_amdgcn_readfirstlane(s_live[kt * NR + j]);
            if (live == 0) continue;
            f32x16 s;
            load_bias(kt, s, (uint32_t)ln * 16);
            Frag vs[2];
            const int ekperm = 16 * (ecol >> 4) + 8 * ((ecol >> 2) & 1) + 4 * ((ecol >> 3) & 1) + (ecol & 3);
            const uint32_t kv = (uint32_t)(ekperm * D + (D > 8 ? 8 * ehf : 0)) * 2, ve = (uint32_t)((ecol < D ? ecol : 0) * 32 + 8 * ehf) * 2;
#pragma unroll
            for (int c = 0; c < 2; ++c) vs[c].u = ldg16(a.vt + off + (size_t)kt * (32 * D) + 16 * c, ve);      // (rows D .. 31 of the context: unused)
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                Frag k;
                k.u = ldg16(a.k + off + (size_t)kt * (32 * D) + 16 * i, kv);
                s = mfma(k.v, qs[i].v, s);
            }
            general_tile(s, vs, live, ehf, o, m, l);
        }
        uint2 gr[D / 8];
        load_gate(r, gr);
        finish(o, l + other_half(l), r, gr);
    }
}

template <int D, int NR, int NW, bool HAS_BIAS>
static ff_status launch(AttnRowsArgs a, hipStream_t st) {
    const int nt = (a.L + 31) / 32;
    const size_t smem = (size_t)(ring_of(NW) + (D < 32 ? 1 : 0)) * NR * 128 * D + (size_t)((nt + 1) & ~1) * NR * 4;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_rows<D, NR, NW, HAS_BIAS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
    if (attr != hipSuccess) return fail(FF_EHIP, "k_attn_rows: dynamic LDS limit: %s", hipGetErrorString(attr));
    a.n_qb = (nt + NW - 1) / NW;
    a.n_rb = (a.rows + NR - 1) / NR;
    a.n_items = a.n_qb * a.n_rb * a.H;
    hipLaunchKernelGGL((k_attn_rows<D, NR, NW, HAS_BIAS>), dim3((a.n_items + 7) / 8 * 8), dim3(NW * 64), smem, st, a);
    return FF_OK;
}

template <int D>
static ff_status launch_d(const AttnRowsArgs& a, hipStream_t st) {
    // Four rows per wavefront share a bias tile four ways.  Two rows where four would leave compute units with fewer than two
    // blocks (128 x 128 triangle attention, the whole call: 32.5 us with four, 29.5 with two; 8 x 300 row attention: 43.8,
    // 40.9), and where there is no bias to share and the registers matter more (attn_rows_waves).
    //
    // Up to 64 positions a row has one or two query tiles: blocks of two wavefronts and two rows, instead of four of which half hold
    // no queries (kernel time of column attention, 64 x 1024 at d = 32: 43.0 -> 33.9 us, 64 x 384 at d = 8: 12.6 -> 8.1; 512 x 64 row
    // attention 22.9 -> 20.1).
    const int nt = (a.L + 31) / 32;
    if (nt <= 2) return a.bias ? launch<D, 2, 2, true>(a, st) : launch<D, 2, 2, false>(a, st);
    const bool few = (int64_t)((nt + 3) / 4) * ((a.rows + 3) / 4) * a.H < 2 * compute_units();
    if (a.bias) return few ? launch<D, 2, 4, true>(a, st) : launch<D, 4, 4, true>(a, st);
    return launch<D, 2, 4, false>(a, st);                     // (at d = 32: 166 registers, three wavefronts per SIMD; four rows: 220, two)
}

ff_status attn_rows_launch(const AttnRowsArgs& a, int d, hipStream_t st) {
    if (d == 8) return launch_d<8>(a, st);
    if (d == 16) return launch_d<16>(a, st);
    return launch_d<32>(a, st);
}

}  // namespace ff
