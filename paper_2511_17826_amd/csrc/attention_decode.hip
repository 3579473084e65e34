// Attention of few queries per sequence (decode steps) for gfx950: the arithmetic of attention_kernel, its bits included,
// with the work of a key tile spread over the wavefronts of a workgroup instead of over its query rows.
//
// attention_kernel gives a wavefront 32 query rows and lets it run scores -> softmax step -> product tile after tile; a
// decode step fills one row of 32 and that chain, 1.3 us per tile, is all a compute unit does.  Here a workgroup owns one
// key/value head of one sequence (or one split of its keys) with up to 16 (query, head) rows in the 16 columns of
// v_mfma_f32_16x16x32, and 12 wavefronts in two roles work on four tiles at a time (a round):
//   * score wavefronts 0..7: wavefront w forms S^T of keys 32 kb .. 32 kb + 31 (kb = w / 4) of tile w % 4: eight matrix
//     instructions, scale, mask, the maximum over its keys; then (barrier A: every half tile's maximum is known) the
//     running maximum in tile order, the weights p, their sum and the weights rounded to 16 bits, which go to LDS;
//   * product wavefronts 8..11 (one per SIMD): wavefront 8 + db keeps o for channels 32 db .. 32 db + 31 and runs the only
//     chain there really is, o = o a + V^T P^T tile after tile, one round behind the scores.
// What makes this exact: the maximum is associative; a tile's scores and weights depend on earlier tiles through the
// running maximum alone; the sum of a tile's weights is handed from lane to lane and wavefront to wavefront so that it is
// added up in the same order; a matrix instruction's columns do not influence each other; and one 16x16x32 instruction
// folds its products in eight consecutive k at a time in ascending order, as two chained 32x32x16 instructions do
// (0 differing bits in 51 million outputs over operands and accumulators spread over tens of binades, both formats).
// K (two rounds ahead) and V (one) are fetched into registers, whole rows at a time, and turned around in
// wavefront-private LDS.  Bound: many sequences, HBM; few, what one compute unit takes in (see plan_decode; 48 bytes/ns for a lone
// sequence of 4096 keys) and the two barriers of a round (1.1 us per round without any load).  One barrier a round, the next
// round's scores formed beside this one's weights, was 0.96 .. 1.07 of the time from 4096 keys on and 1 us slower up to 1024:
// intake it is.  K fragments loaded straight into the matrix instruction's layout (no LDS, 64 bytes of 16 rows per load)
// were slower: 47 instead of 34 us below.
// Measured, 32 query heads over 8, bf16, time of a call on the stream, attention_kernel -> this kernel: 1 x 4096 keys
// 90 -> 28 us, 6 sequences of 96 .. 4001 keys 89 -> 28 us, 16 x 4096 98 -> 56 us (4.8 TB/s of K + V), 64 x 4096
// 202 -> 194 us (5.5 TB/s), 1 x 32768 98 -> 49 us, 80 x 10000 786 -> 606 us; 40 heads over 8 (groups of five, which
// attention_kernel does not pack), 16 x 4096 233 -> 70 us.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "attention_common.hpp"

namespace tbik {

constexpr int DEC_ROUND = 4;                                      // key tiles per round
constexpr int DEC_SCORE_WAVES = 2 * DEC_ROUND, DEC_PROD_WAVES = ATT_D / 32;
constexpr int DEC_THREADS = 64 * (DEC_SCORE_WAVES + DEC_PROD_WAVES);
constexpr int DEC_COLS = 16;                                      // (query, head) rows of a workgroup
static_assert(ATT_SPLIT % DEC_ROUND == 0, "a round does not cross a split");
// LDS map (bytes)
constexpr int DEC_V_TILE = ATT_KV * 32 * 2;                       // a product wavefront's channels of a tile
constexpr int DEC_P_ROUND = DEC_ROUND * 2 * 64 * 16;              // a round's weights, as B fragments of 32 keys
constexpr int DEC_K_WAVE = 32 * ATT_D * 2;                        // a score wavefront's half tile
constexpr int DEC_LDS_V = DEC_SCORE_WAVES * DEC_K_WAVE;
constexpr int DEC_LDS_P = DEC_LDS_V + DEC_PROD_WAVES * 2 * DEC_V_TILE;
constexpr int DEC_LDS_PMAX = DEC_LDS_P + 2 * DEC_P_ROUND;
constexpr int DEC_LDS_HSUM = DEC_LDS_PMAX + 2 * DEC_SCORE_WAVES * DEC_COLS * 4;
constexpr int DEC_LDS_PSUM = DEC_LDS_HSUM + 2 * DEC_ROUND * 32 * 4;
static_assert(DEC_V_TILE == DEC_ROUND * 1024, "the first four wavefronts fill a tile");
constexpr int DEC_LDS_ZERO = DEC_LDS_PSUM + 2 * DEC_ROUND * DEC_COLS * 4;    // a tile of values that are -0
constexpr int DEC_LDS = DEC_LDS_ZERO + DEC_V_TILE;
static_assert(DEC_LDS <= 160 * 1024, "LDS of a compute unit");
// A split's state: chunk c of lane t at [c * 64 + t] of 16 bytes; chunk 0 is (m, l, -, -), chunk 1 + 2 db + bl holds the
// lane's four channels of o in the bl-th 16 of channel block db.
constexpr int DEC_STATE_CHUNKS = (1 + ATT_D / 16) * 64;

struct DecodeParams {
    const uint16_t *Q, *K, *V;
    uint16_t *O;
    const int32_t *cu_q, *cu_k;
    int64_t q_stride, k_stride, v_stride, o_stride;               // token strides, elements
    int total_q, total_k;
    int group, rows;                                              // query heads per key/value head; columns per head
    int heads_kv, col_groups;                                     // col_groups: workgroups that share the rows of a head, 16 each
    int n_splits;                                                 // 1: a workgroup walks all splits, folding as it goes
    int items, chan_groups;                                       // (sequence, split, column group, kv head) items; workgroups per item
    int max_tiles;                                                // key tiles of a sequence of max_seqlen_k keys
    float c;                                                      // scale * log2(e)
    f32x4 *states;                                                // n_splits > 1: [sequence][kv head][split]
};

typedef __attribute__((address_space(1))) const char dec_gchar;
typedef __attribute__((address_space(1))) const att_u32x4 dec_gvec;

__device__ __forceinline__ void workgroup_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <bool F16>
__device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// v_permlane16_swap of (v, v): rows of 16 lanes (r0, r0, r2, r2) and (r1, r1, r3, r3).
__device__ __forceinline__ void both_rows(float v, float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// (m2, l2, o2) <- fold of the earlier splits' state (m2, l2, o2) and the next split's (m, l, o): the operations of
// attention_kernel's state_fold, each rounded once; an empty state is skipped exactly.
__device__ __forceinline__ void fold_states(float &m2, float &l2, f32x4 (&o2)[2], float m, float l, const f32x4 (&o)[2]) {
    const float M = fmaxf(m2, m);
    const float m_use = (M == -INFINITY) ? 0.0f : M;
    const float a2 = __builtin_amdgcn_exp2f(m2 - m_use), a1 = __builtin_amdgcn_exp2f(m - m_use);
    const bool next_empty = (l == 0.0f), so_far_empty = (l2 == 0.0f);
#pragma unroll
    for (int bl = 0; bl < 2; ++bl)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float t = __fadd_rn(__fmul_rn(o2[bl][i], a2), __fmul_rn(o[bl][i], a1));
            o2[bl][i] = next_empty ? o2[bl][i] : (so_far_empty ? o[bl][i] : t);
        }
    const float lt = __fadd_rn(__fmul_rn(l2, a2), __fmul_rn(l, a1));
    l2 = next_empty ? l2 : (so_far_empty ? l : lt);
    m2 = next_empty ? m2 : (so_far_empty ? m : M);
}

// O = o / l for a lane's channels (16 bl + 4 g .. + 3 of a block of 32, optr at 4 g), one rounding.
template <bool F16>
__device__ __forceinline__ void store_channels(uint16_t *optr, float l, const f32x4 (&o)[2]) {
#pragma unroll
    for (int bl = 0; bl < 2; ++bl) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (l > 0.0f) ? o[bl][i] / l : 0.0f;
        att_u32x2 w;
        w[0] = pack_16x2<F16>(v[0], v[1]);
        w[1] = pack_16x2<F16>(v[2], v[3]);
        *reinterpret_cast<att_u32x2 *>(optr + 16 * bl) = w;
    }
}

// A workgroup's part of the work: key/value head, rows 16 cg .. + 15 of it, and the split (n_splits > 1) of sequence seq.
struct DecodeItem {
    int hk, cg, seq, split, n_splits;
    int q0, Lq, k0, Lk;                                           // the sequence's queries and keys in the packed tensors
    int first_block, my_blocks;                                   // channel blocks of the values
};

// Queries q_base .. q_base + rows - 1 of an item.
template <bool CAUSAL, bool F16>
__device__ __forceinline__ void decode_queries(const DecodeParams &p, const DecodeItem &it, int q_base, int tid, unsigned char *smem) {
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int q0 = it.q0, k0 = it.k0, Lq = it.Lq, Lk = it.Lk, hk = it.hk;
    const int shift = Lk - Lq;                                    // the queries are the last Lq positions
    const int q_last = min(Lq, q_base + p.rows) - 1;
    const int lim_block = CAUSAL ? min(Lk - 1, q_last + shift) : Lk - 1;
    const int n_tiles = lim_block >= 0 ? min(p.max_tiles, lim_block / ATT_KV + 1) : 0;   // keys past max_seqlen_k are left out

    // This lane's row: column col is query q_base + col % rows of head col / rows of the group; columns past those repeat one.
    const int col = it.cg * DEC_COLS + l16;
    const int head = hk * p.group + min(col / p.rows, p.group - 1), qrow = q_base + col % p.rows;
    const bool stored = col < p.group * p.rows && qrow < Lq;
    const int qpos = min(qrow, Lq - 1);
    const int lim = CAUSAL ? min(Lk - 1, qpos + shift) : Lk - 1;  // last visible key; < 0: none
    const int full = CAUSAL ? min(Lk - 1, q_base + shift) : Lk - 1;        // last key that every row sees

    const int t_begin = it.n_splits > 1 ? it.split * ATT_SPLIT : 0;
    const int t_end = it.n_splits > 1 ? min(n_tiles, t_begin + ATT_SPLIT) : n_tiles;
    f32x4 *const state = p.states + (((size_t)(it.seq * p.col_groups + it.cg) * p.heads_kv + hk) * p.n_splits + it.split) * DEC_STATE_CHUNKS + lane;
    const int db = wave < DEC_SCORE_WAVES ? 0 : it.first_block + wave - DEC_SCORE_WAVES;   // a product wavefront's channel block
    if (t_begin >= t_end) {                                       // uniform: no row sees a key (of this split)
        if (wave < DEC_SCORE_WAVES) return;
        if (it.n_splits > 1) {
            if (db == 0) state[0] = f32x4{-INFINITY, 0.0f, 0.0f, 0.0f};         // an empty state: only m and l are looked at
        } else if (stored) {
            const f32x4 zero[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
            store_channels<F16>(p.O + (int64_t)(q0 + qrow) * p.o_stride + (int64_t)head * ATT_D + db * 32 + 4 * g4, 0.0f, zero);
        }
        return;
    }
    const int key_end = min(Lk, t_end * ATT_KV);                  // > 0: the keys of this workgroup end here
    const int rounds = (t_end - t_begin + DEC_ROUND - 1) / DEC_ROUND;
    float *const pmax = reinterpret_cast<float *>(smem + DEC_LDS_PMAX);
    float *const hsum = reinterpret_cast<float *>(smem + DEC_LDS_HSUM);
    float *const psum = reinterpret_cast<float *>(smem + DEC_LDS_PSUM);
    constexpr int ROUNDS_PER_SPLIT = ATT_SPLIT / DEC_ROUND;

    if (wave < DEC_SCORE_WAVES) {
        // ------------------------------------------------------------------ scores
        const int qt = wave & (DEC_ROUND - 1), kb = wave / DEC_ROUND;
        bf16x8 bq[ATT_D / 32];                                    // Q^T: column l16, channels 32 ks + 8 g4 .. + 7
        {
            const uint16_t *qptr = p.Q + (int64_t)(q0 + qpos) * p.q_stride + (int64_t)head * ATT_D + g4 * 8;
#pragma unroll
            for (int ks = 0; ks < ATT_D / 32; ++ks) bq[ks] = *reinterpret_cast<const bf16x8 *>(qptr + ks * 32);
        }
        dec_gchar *const kbase = (dec_gchar *)(p.K + (int64_t)k0 * p.k_stride + (int64_t)hk * ATT_D);
        const int row_bytes = (int)p.k_stride * 2;
        // Half tile of keys: load i brings rows 4 i .. 4 i + 3, 16 lanes a row.  Unconditional, as everything in the loops
        // below: a load behind a branch makes the compiler wait for all loads in flight where the paths meet.  Past the end
        // the last key is fetched again (it is masked), at one place of the cache.
        const int sub = lane >> 4, pos = lane & 15, sub_bytes = sub * row_bytes;
        auto load_k = [&](att_u32x4 (&kr)[8], int t) __attribute__((always_inline)) {
            const int key0 = min(t * ATT_KV + kb * 32, key_end - 1), last = min(key_end - 1 - key0, 31) * row_bytes;   // uniform
            dec_gchar *const base = kbase + (int64_t)key0 * row_bytes;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                kr[i] = *(dec_gvec *)(base + (uint64_t)(uint32_t)(min(sub_bytes + 4 * i * row_bytes, last) + pos * 16));
        };
        unsigned char *const k_lds = smem + wave * DEC_K_WAVE;    // chunk c of row r sits at position c ^ (r & 15)
        unsigned char *const k_wr = k_lds + sub * 256;
        const int wr_pos = (pos ^ sub) << 4;
        const unsigned char *const k_rd = k_lds + l16 * 256;
        unsigned char *const p_wr = smem + DEC_LDS_P + (qt * 2 + kb) * 1024 + lane * 16;

        if (wave < DEC_ROUND)                                     // (+0 x -0 = -0, and x + -0 is x for either zero; past barrier A of round 0)
            *reinterpret_cast<att_u32x4 *>(smem + DEC_LDS_ZERO + wave * 1024 + lane * 16) = att_u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};

        float m = -INFINITY;
        auto round = [&](att_u32x4 (&kr)[8], int r) __attribute__((always_inline)) {
            const int t = t_begin + r * DEC_ROUND + qt, b = r & 1;
            if (r > 0 && r % ROUNDS_PER_SPLIT == 0) m = -INFINITY;        // a split begins (walking form)
            // A tile past the end (the last round may have some) is one that no row sees: its maximum is -inf, its weights 0.
#pragma unroll
            for (int i = 0; i < 8; ++i) *reinterpret_cast<att_u32x4 *>(k_wr + i * 1024 + (wr_pos ^ ((4 * i & 12) << 4))) = kr[i];
            load_k(kr, t + 2 * DEC_ROUND);
            f32x4 s[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};            // keys 16 j + 4 g4 + i of the half tile
#pragma unroll
            for (int ks = 0; ks < ATT_D / 32; ++ks)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    s[j] = mfma_16x16x32<F16>(*reinterpret_cast<const bf16x8 *>(k_rd + j * 4096 + (((4 * ks + g4) ^ l16) << 4)), bq[ks], s[j]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[j][i] = s[j][i] * p.c;
            if (t * ATT_KV + kb * 32 + 31 > full) {               // uniform: some row does not see the whole half tile
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (t * ATT_KV + kb * 32 + 16 * j + 4 * g4 + i > lim) s[j][i] = -INFINITY;
            }
            float tmax = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
            float a, c;
            both_halves(tmax, a, c);
            tmax = fmaxf(a, c);
            both_rows(tmax, a, c);
            if (lane < DEC_COLS) pmax[(b * DEC_SCORE_WAVES + wave) * DEC_COLS + lane] = fmaxf(a, c);
            workgroup_barrier();                                  // A
            float m_mine = m;
#pragma unroll
            for (int q = 0; q < DEC_ROUND; ++q) {
                const float *pm = pmax + (b * DEC_SCORE_WAVES + q) * DEC_COLS + l16;
                m = fmaxf(m, fmaxf(pm[0], pm[DEC_ROUND * DEC_COLS]));
                if (q == qt) m_mine = m;
            }
            const float m_use = (m_mine == -INFINITY) ? 0.0f : m_mine;      // a row that has seen no key yet
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[j][i] = __builtin_amdgcn_exp2f(s[j][i] - m_use);
            // The two halves of the wavefront swap: afterwards a lane's eight weights are those of keys 16 h + 4 g .. + 3 and
            // 16 h + 8 + 4 g .. + 3 (g4 = 2 h + g): k-slots 8 g4 .. 8 g4 + 7 of the product's instruction, in the order of
            // attention_kernel's two steps.
            float w[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const auto r2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[0][i]), __float_as_uint(s[1][i]), false, false);
                w[i] = __uint_as_float(r2[0]);
                w[4 + i] = __uint_as_float(r2[1]);
            }
            {
                att_u32x4 pk;
#pragma unroll
                for (int i = 0; i < 4; ++i) pk[i] = pack_16x2<F16>(w[2 * i], w[2 * i + 1]);
                *reinterpret_cast<att_u32x4 *>(p_wr + b * DEC_P_ROUND) = pk;
            }
            // Sum of the tile's weights, per g: the eight of h = 0, then those of h = 1, then the other wavefront's 32 keys.
            auto add_own = [&](float sum) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 8; ++i) sum = sum + w[i];     // right in the lower half of the wavefront ...
                both_halves(sum, a, c);
                sum = a;
#pragma unroll
                for (int i = 0; i < 8; ++i) sum = sum + w[i];     // ... and now in the upper one
                return sum;
            };
            if (kb == 0) {
                const float sum = add_own(0.0f);
                if (lane >= 32) hsum[(b * DEC_ROUND + qt) * 32 + lane - 32] = sum;
            }
            workgroup_barrier();                                  // B
            if (kb == 1) {
                const float sum = add_own(hsum[(b * DEC_ROUND + qt) * 32 + (lane & 31)]);
                both_rows(sum, a, c);
                if (g4 == 2) psum[(b * DEC_ROUND + qt) * DEC_COLS + l16] = a + c;
            }
        };
        att_u32x4 kr0[8], kr1[8];
        load_k(kr0, t_begin + qt);
        load_k(kr1, t_begin + DEC_ROUND + qt);
        for (int r = 0; r + 1 < rounds; r += 2) {                 // (no way out between the two: see load_k)
            round(kr0, r);
            round(kr1, r + 1);
        }
        if (rounds & 1) round(kr0, rounds - 1);
        workgroup_barrier();                                      // A of the round that is not there: the last sums are written
        return;
    }

    // ---------------------------------------------------------------------- product
    const int sub = lane >> 2, pos = lane & 3;                    // load i of a tile brings keys 16 i .. 16 i + 15, 4 lanes a key
    dec_gchar *const vbase = (dec_gchar *)(p.V + (int64_t)k0 * p.v_stride + (int64_t)hk * ATT_D + db * 32);
    const int row_bytes = (int)p.v_stride * 2;
    const int sub_bytes = sub * row_bytes;
    auto load_v = [&](att_u32x4 (&vr)[4], int t) __attribute__((always_inline)) {
        const int key0 = min(t * ATT_KV, key_end - 1), last = min(key_end - 1 - key0, ATT_KV - 1) * row_bytes;
        dec_gchar *const base = vbase + (int64_t)key0 * row_bytes;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            vr[i] = *(dec_gvec *)(base + (uint64_t)(uint32_t)(min(sub_bytes + 16 * i * row_bytes, last) + pos * 16));
    };
    // A key's 32 channels are 64 bytes in LDS, the two halves of 16 channels exchanged in keys 4 .. 7 of every 8: a
    // transposing read's 16 lanes take 4 keys x 16 channels, and the two groups that read keys 0 .. 3 and 4 .. 7 then hit
    // different banks.
    const int g = g4 & 1;
    unsigned char *const v_wr = smem + DEC_LDS_V + (wave - DEC_SCORE_WAVES) * 2 * DEC_V_TILE + sub * 64 + ((pos ^ (2 * g)) << 4);           // (sub >> 2) & 1 == g4 & 1
    const unsigned char *const v_rd = smem + (16 * (g4 >> 1) + 4 * g + (l16 >> 2)) * 64 + (l16 & 3) * 8;       // + the tile's place
    const int v_at = DEC_LDS_V + (wave - DEC_SCORE_WAVES) * 2 * DEC_V_TILE;
    const unsigned char *const p_rd = smem + DEC_LDS_P + lane * 16;

    att_u32x4 vr[DEC_ROUND][4];
#pragma unroll
    for (int q = 0; q < DEC_ROUND; ++q) load_v(vr[q], t_begin + q);

    f32x4 o[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};                    // channels 32 db + 16 bl + 4 g4 + i
    f32x4 o_acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};                // the folded splits before this one
    float m_acc = -INFINITY, l_acc = 0.0f;
    float m = -INFINITY, l = 0.0f, alpha[DEC_ROUND];

    // Tiles q and q + 1 of round r: V through LDS, then o = o alpha + V^T P^T tile after tile.
    auto two_tiles = [&](auto q_tag, int r) __attribute__((always_inline)) {
        constexpr int Q0 = decltype(q_tag)::value;
#pragma unroll
        for (int q = Q0; q < Q0 + 2; ++q) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<att_u32x4 *>(v_wr + (q & 1) * DEC_V_TILE + i * 1024) = vr[q][i];
            load_v(vr[q], t_begin + (r + 1) * DEC_ROUND + q);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            // A tile past the end (the last round may have some) leaves o as it is: its weights are 0, its values must be finite.
            // (Values replaced in registers, or behind a branch in LDS, cost 5 and 3 % where most rounds are the last.)
            const unsigned char *const rd = v_rd + (t_begin + r * DEC_ROUND + Q0 + u < t_end ? v_at + u * DEC_V_TILE : DEC_LDS_ZERO);   // uniform
            bf16x8 pb[2];
            union { att_v4i16 h2[2]; bf16x8 v; } vf[2][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                pb[kb] = *reinterpret_cast<const bf16x8 *>(p_rd + (r & 1) * DEC_P_ROUND + ((Q0 + u) * 2 + kb) * 1024);
#pragma unroll
                for (int bl = 0; bl < 2; ++bl)
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh)
                        vf[kb][bl].h2[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (__attribute__((address_space(3))) att_v4i16 *)(rd + (32 * kb + 8 * hh) * 64 + ((bl ^ g) << 5)));
            }
#pragma unroll
            for (int bl = 0; bl < 2; ++bl)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[bl][i] = o[bl][i] * alpha[Q0 + u];       // o * 1 is o
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int bl = 0; bl < 2; ++bl) o[bl] = mfma_16x16x32<F16>(vf[kb][bl].v, pb[kb], o[bl]);
        }
    };
    // What is left of round r once the sums of its weights are there (past barrier A of the next round).
    auto finish_round = [&](int r) __attribute__((always_inline)) {
        two_tiles(std::integral_constant<int, 2>{}, r);
#pragma unroll
        for (int q = 0; q < DEC_ROUND; ++q) l = l * alpha[q] + psum[((r & 1) * DEC_ROUND + q) * DEC_COLS + l16];
    };
    for (int r = 0; r < rounds; ++r) {
        workgroup_barrier();                                      // A
        if (r > 0) {
            finish_round(r - 1);
            if (r % ROUNDS_PER_SPLIT == 0) {                      // a split ends here (walking form)
                fold_states(m_acc, l_acc, o_acc, m, l, o);
                o[0] = o[1] = f32x4{0, 0, 0, 0};
                m = -INFINITY;
                l = 0.0f;
            }
        }
        workgroup_barrier();                                      // B
#pragma unroll
        for (int q = 0; q < DEC_ROUND; ++q) {
            const float *pm = pmax + ((r & 1) * DEC_SCORE_WAVES + q) * DEC_COLS + l16;
            const float m_new = fmaxf(m, fmaxf(pm[0], pm[DEC_ROUND * DEC_COLS]));
            const float m_use = (m_new == -INFINITY) ? 0.0f : m_new;      // a row that has seen no key yet
            alpha[q] = __builtin_amdgcn_exp2f(m - m_use);
            m = m_new;
        }
        two_tiles(std::integral_constant<int, 0>{}, r);
    }
    workgroup_barrier();
    finish_round(rounds - 1);

    if (it.n_splits > 1) {                                        // the state as it is; attention_decode_merge_kernel folds and divides
        if (db == 0) state[0] = f32x4{m, l, 0.0f, 0.0f};
        state[(1 + 2 * db) * 64] = o[0];
        state[(2 + 2 * db) * 64] = o[1];
        return;
    }
    fold_states(m_acc, l_acc, o_acc, m, l, o);                    // one split only: the accumulated state is empty
    if (stored) store_channels<F16>(p.O + (int64_t)(q0 + qrow) * p.o_stride + (int64_t)head * ATT_D + db * 32 + 4 * g4, l_acc, o_acc);
}

template <bool CAUSAL, bool F16>
__global__ __launch_bounds__(DEC_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3)))
void attention_decode_kernel(const DecodeParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // Workgroups of one item -- the same keys, different channels of the values -- follow each other on one XCD.
    int id = (int)(blockIdx.x >> 3) / p.chan_groups * 8 + (blockIdx.x & 7);
    if (id >= p.items) return;
    DecodeItem it;
    it.my_blocks = ATT_D / 32 / p.chan_groups;
    it.first_block = (int)(blockIdx.x >> 3) % p.chan_groups * it.my_blocks;
    if (wave >= DEC_SCORE_WAVES + it.my_blocks) return;
    it.hk = id % p.heads_kv;
    id /= p.heads_kv;
    it.cg = id % p.col_groups;
    id /= p.col_groups;
    it.n_splits = p.n_splits;
    it.split = id % p.n_splits;
    it.seq = id / p.n_splits;

    // Sequence bounds, clamped so that no value of the offset arrays can lead outside the tensors.
    it.q0 = clampi(p.cu_q[it.seq], 0, p.total_q);
    it.Lq = clampi(p.cu_q[it.seq + 1], it.q0, p.total_q) - it.q0;
    it.k0 = clampi(p.cu_k[it.seq], 0, p.total_k);
    it.Lk = clampi(p.cu_k[it.seq + 1], it.k0, p.total_k) - it.k0;
    if (it.Lq <= 0) return;                                       // uniform
    decode_queries<CAUSAL, F16>(p, it, 0, threadIdx.x, smem);
    // A sequence with more queries than max_seqlen_q said (the host does not know): one workgroup walks the splits for the
    // rest of them.  (A second copy of the code: one copy in a loop spills 41 registers.)
    if (it.split != 0) return;
    it.n_splits = 1;
    for (int q_base = p.rows; q_base < it.Lq; q_base += p.rows) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid), "+s"(it.Lk), "+s"(it.k0), "+s"(it.hk));     // nothing is computed before the loop and kept in registers
        workgroup_barrier();                                      // the LDS of the queries before these has been read
        decode_queries<CAUSAL, F16>(p, it, q_base, tid, smem);
    }
}

// Folds the states of a (sequence, column group, key/value head)'s splits in ascending order and writes the output;
// wavefront db takes channels 32 db .. 32 db + 31.  The states of eight splits are fetched at a time.
template <bool F16>
__global__ __launch_bounds__(64 * DEC_PROD_WAVES) void attention_decode_merge_kernel(const DecodeParams p) {
    const int lane = threadIdx.x & 63, db = threadIdx.x >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int hk = blockIdx.x % p.heads_kv, cg = blockIdx.x / p.heads_kv % p.col_groups, seq = blockIdx.x / p.heads_kv / p.col_groups;
    const int q0 = clampi(p.cu_q[seq], 0, p.total_q), q1 = clampi(p.cu_q[seq + 1], q0, p.total_q);
    const int Lq = q1 - q0;
    const int col = cg * DEC_COLS + l16;
    const int head = hk * p.group + min(col / p.rows, p.group - 1), qrow = col % p.rows;
    if (col >= p.group * p.rows || qrow >= Lq) return;
    const f32x4 *states = p.states + (size_t)blockIdx.x * p.n_splits * DEC_STATE_CHUNKS + lane;
    float m = -INFINITY, l = 0.0f;
    f32x4 o[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    constexpr int AHEAD = 8;
    for (int j0 = 0; j0 < p.n_splits; j0 += AHEAD) {
        f32x4 h[AHEAD], x[AHEAD][2];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const f32x4 *st = states + (size_t)min(j0 + u, p.n_splits - 1) * DEC_STATE_CHUNKS;
            h[u] = st[0];
            x[u][0] = st[(1 + 2 * db) * 64];
            x[u][1] = st[(2 + 2 * db) * 64];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (j0 + u < p.n_splits && h[u][1] != 0.0f)           // (an empty split's o was never written)
                fold_states(m, l, o, h[u][0], h[u][1], x[u]);
    }
    store_channels<F16>(p.O + (int64_t)(q0 + qrow) * p.o_stride + (int64_t)head * ATT_D + db * 32 + 4 * g4, l, o);
}

// The scratch area of a call stays below this (the bound of attention_kernel's calls).
constexpr size_t DEC_MAX_STATE_BYTES = (size_t)306 << 20;

// One workgroup per split while that leaves the chip short of work; enough sequences walk their splits in registers.  A
// compute unit takes in 53 bytes per ns from HBM while few do and 32 with 192 of them, whether 32 or 256 KiB are under way
// (plain loads of consecutive rows; from the memory-side cache 150 and 39), so while compute units are left over an item's value channels are dealt to two or four workgroups, each of which
// forms all scores: K is fetched once per XCD, and a workgroup reads 3/4 or 5/8 of the bytes.
struct DecodePlan {
    int col_groups, n_splits;
    size_t state_bytes;
};
static DecodePlan plan_decode(int batch, int max_seqlen_q, int max_seqlen_k, int heads_q, int heads_kv) {
    const int splits = max_seqlen_k > 0 ? (max_seqlen_k + ATT_SPLIT * ATT_KV - 1) / (ATT_SPLIT * ATT_KV) : 1;
    const int col_groups = (max_seqlen_q * (heads_q / heads_kv) + DEC_COLS - 1) / DEC_COLS;
    const int64_t items = (int64_t)batch * heads_kv * col_groups;
    const size_t states = (size_t)items * splits * DEC_STATE_CHUNKS * sizeof(f32x4);
    if (splits == 1 || items >= 512 || states > DEC_MAX_STATE_BYTES) return {col_groups, 1, 0};
    return {col_groups, splits, states};
}

// A launch holds fewer than 2^32 threads: from 5.6 million items on, 65535 sequences on 86 key/value heads, these workgroups
// of 768 are too many where attention_kernel's of 256 are not.
static bool launches(int batch, int max_seqlen_q, int heads_q, int heads_kv) {
    return ((int64_t)batch * heads_kv * plan_decode(batch, max_seqlen_q, 0, heads_q, heads_kv).col_groups + 7) / 8 * 8 * DEC_THREADS < ((int64_t)1 << 32);
}

// Where attention_kernel is the quicker one although a sequence has few queries: it has two workgroups on a compute unit
// where this kernel has one, so it is a matter of rounds, and only for groups that it packs into one workgroup (powers of
// two; the others it reads once per query head).  Times of the two, attention_kernel first; the lines were drawn on 8800 shapes
// of 1 .. 10000 keys.  Since then that kernel overlaps its tiles: over 1500 shapes timed again the choice is 0.3 % above the quicker
// kernel in the mean, more than 4 % above it at 46 (24 % at most), most of them on this kernel's side of a line.
//   * More than 16 rows on a key/value head: its keys are read here by two workgroups.  64 heads over 8, 4 queries: 33
//     sequences of 4096 keys 131 / 174 us, 32 of 64 keys 10.0 / 11.1 (16 of them 8.1 / 6.3), 128 of 1024 keys 112 / 155.
//   * One key tile is over before the rounds overlap.  32 heads over 32: 9 sequences of 64 keys 9.5 / 10.1 us, 200 of them
//     91 / 108; two query heads per key/value head lose from 3 rounds on, four from 7 (a tenth at most).  (4 heads over 4: 128
//     sequences 14.0 / 10.8, the neighbours lose as well; left to this kernel.)
//   * Sequences of nearly one length and a second round that is nearly empty.  16 heads over 16: 18 sequences of 2048 keys
//     take 1.14 times the time here, 22 of them 1.09, 28 1.02; 32 heads over 8: 33 of 4096 keys 1.20, 40 of them 1.11, 48
//     1.05 (1.01 when the line was drawn).  With lengths spread over a factor of ten this kernel wins there, by 1.1 to 2.5.
static bool attention_kernel_is_quicker(const AttnArgs &a) {
    const int group = a.heads_q / a.heads_kv;
    if (group & (group - 1)) return false;
    const int64_t heads = (int64_t)a.batch * a.heads_kv;
    if (a.max_seqlen_q * group > DEC_COLS) return heads > (a.max_seqlen_k <= 2 * ATT_KV ? 128 : 256);
    if (a.max_seqlen_k <= ATT_KV) return a.heads_kv >= 8 && heads > 256 * (2 * group - 1);
    if (a.max_seqlen_k < 1024 || a.max_seqlen_k > ATT_SPLIT * ATT_KV || heads <= 256 || 10 * (int64_t)a.total_k < 9 * (int64_t)a.batch * a.max_seqlen_k) return false;
    return group <= 2 ? heads <= (a.max_seqlen_k >= 2048 ? 352 : 288) : group == 4 && a.max_seqlen_k >= 3000 && heads <= 320;
}

bool attention_decode_takes(const AttnArgs &a) {
    return attention_decode_supports(a.max_seqlen_q, a.heads_q, a.heads_kv) && launches(a.batch, a.max_seqlen_q, a.heads_q, a.heads_kv) &&
           !attention_kernel_is_quicker(a);
}

bool attention_decode_supports(int max_seqlen_q, int heads_q, int heads_kv) {
    return (int64_t)max_seqlen_q * (heads_q / heads_kv) <= 2 * DEC_COLS;
}

size_t attention_decode_workspace(int batch, int max_seqlen_q, int max_seqlen_k, int heads_q, int heads_kv) {
    return plan_decode(batch, max_seqlen_q, max_seqlen_k, heads_q, heads_kv).state_bytes;
}

template <bool F16>
static hipError_t launch_decode_of(const AttnArgs &a, const DecodeParams &p, hipStream_t s) {
    static std::atomic<unsigned> done[2] = {{0}, {0}};            // bit d: the LDS attribute is set on device d
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) dev = 32;      // 32: not remembered, set every time
    auto kernel = a.causal ? attention_decode_kernel<true, F16> : attention_decode_kernel<false, F16>;
    std::atomic<unsigned> &flag = done[a.causal ? 0 : 1];
    if (dev >= 32 || !((flag.load(std::memory_order_relaxed) >> dev) & 1u)) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, DEC_LDS);
        if (e != hipSuccess) return e;
        if (dev < 32) flag.fetch_or(1u << dev, std::memory_order_relaxed);
    }
    const unsigned items = (unsigned)(a.batch * a.heads_kv * p.col_groups);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((p.items + 7) / 8 * 8 * p.chan_groups)), dim3(DEC_THREADS), DEC_LDS, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.n_splits == 1) return e;
    hipLaunchKernelGGL(attention_decode_merge_kernel<F16>, dim3(items), dim3(64 * DEC_PROD_WAVES), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_attention_decode(const AttnArgs &a, hipStream_t s) {
    DecodePlan pl = plan_decode(a.batch, a.max_seqlen_q, a.max_seqlen_k, a.heads_q, a.heads_kv);
    // A workspace of the size that attention_kernel asks for may not hold the states; walking needs none and has the same bits.
    // (Where that kernel would have the splits side by side its 68 KiB per state and split are room enough for these 9 KiB.)
    if (pl.state_bytes > (a.workspace ? a.workspace_bytes : 0)) pl.n_splits = 1;
    DecodeParams p;
    p.Q = a.Q; p.K = a.K; p.V = a.V; p.O = a.O;
    p.cu_q = a.cu_q; p.cu_k = a.cu_k;
    p.q_stride = a.q_stride; p.k_stride = a.k_stride; p.v_stride = a.v_stride; p.o_stride = a.o_stride;
    p.total_q = a.total_q; p.total_k = a.total_k;
    p.group = a.heads_q / a.heads_kv;
    p.rows = a.max_seqlen_q;
    p.heads_kv = a.heads_kv;
    p.col_groups = pl.col_groups;
    p.n_splits = pl.n_splits;
    p.items = a.batch * a.heads_kv * pl.col_groups * pl.n_splits;
    p.chan_groups = p.items <= 64 ? 4 : p.items <= 128 ? 2 : 1;
    p.max_tiles = a.max_seqlen_k > 0 ? (a.max_seqlen_k + ATT_SPLIT * ATT_KV - 1) / (ATT_SPLIT * ATT_KV) * ATT_SPLIT : ATT_SPLIT;
    p.c = a.scale * 1.44269504088896340736f;
    p.states = reinterpret_cast<f32x4 *>(a.workspace);
    return a.dtype == TBIK_F16 ? launch_decode_of<true>(a, p, s) : launch_decode_of<false>(a, p, s);
}

}  // namespace tbik
