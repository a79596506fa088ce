// Paged attention for bf16 caches, head_dim 128, 16-position pages, decode form: the layer's
// HBM-bound operator (the paper's memory-bound "decode attention", Section 2).  The work lists it shares
// with the prefill form (kernels_attn_prefill.hip) are kernels_attn_plan.hip's.
//
// A wave serves one token of a single-token sequence against one chunk (up to the handle's
// chunk size, 256 positions by default; a sequence's chunks are of equal size up to rounding) of one kv head, all q heads of that kv head's group at once, so K and V are fetched once per kv
// head.  A page of K is 16 rows of 256 bytes, a page of V is 128 rows (one per head-dim
// index) of 32 bytes; both are loaded straight into MFMA operand layout with fully used
// 64-byte / 32-byte row segments, no LDS.  The group's scores are a skinny but real
// contraction
//     S[16 positions, G heads] = K_page[16, 128] Q^T[128, G]      (4 x mfma 16x16x32)
//     O^T[128, G]           += V_page^T[128, 16] P[16, G]         (8 x mfma 16x16x16)
// whose D layout (lane: head l%16, positions 4*(l/16)+r) is exactly the B layout the second
// product wants, so probabilities never cross lanes.  Doing the same dot products on the
// vector ALUs would need about 28 wave instructions per cached position and kv head, which
// at HBM rate is most of the ALU issue slots of a CU; on the matrix cores it is a few
// percent.  Softmax is online per tile of two pages in the exp2 domain with the running
// max shared by the four lanes of a head; the partial (m, l, o) of the chunk goes to the
// split-KV arrays and attn_combine_kernel merges chunks in order.
#include <algorithm>

#include "attn_prefill.h"
#include "common.h"
#include "kernels.h"

namespace dyn {

hipError_t launch_attention_combine(int dtype, bool base2, float *part_o, float *part_ml,
                                    const int32_t *pos_of_token, const int32_t *ct_of_token, void *out, int ld_out,
                                    const AttnShape &sh, int rows, hipStream_t s, int32_t *counter_reset, bool one_chunk_done);
hipError_t launch_attention_prefill(const void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                                    const int32_t *block_table, const void *k_cache, const void *v_cache, void *out, int ld_out,
                                    float *part_o, float *part_ml, const AttnShape &sh, int32_t *plan, const int32_t *ct_of_token, long max_items, int max_groups,
                                    hipStream_t s);

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int HD = 128, PS = 16, TILE_PAGES = 2;
constexpr int kPersistentGroups = 512;   // two 4-wave workgroups for each of the 256 CUs

// Persistent waves: in round k wave w of the launch (numbered by gw below) takes (entry, kv head) pair k * n_waves + w,
// in odd rounds k * n_waves + (n_waves - 1 - w): a snake over a list that is ordered largest first
// (attn_plan_kernel), so a wave that drew the largest item of one round draws the smallest of the next.
// A pair is walked two tiles (four pages) at a time through two register buffers, and when a
// pair runs out of tiles the free buffer is refilled with the first tile of the wave's next
// pair - whose indices were fetched while this pair was being multiplied - so the stream of
// loads never drains at a pair boundary and the three dependent lookups (work list ->
// position / sequence -> block table) are off the critical path.
// NQG = sets of 16 MFMA columns per wave; the decode list uses 1 (eight waves per CU keep HBM
// busy, 4 of the 16 columns live with four q heads per kv head).
struct AttnItem {
    int t, c, n_tok;                  // first token row of the query group, chunk, tokens in the group
    int n_keys, lp_first, seq_pages;  // keys the group's last token attends, first logical page of the chunk, the sequence's pages
    int lp_last, key_end;             // last logical page of the chunk; first position past the chunk (at most n_keys)
    int n_pair;                       // tile pairs to walk
    const int32_t *bt;                // block-table row of the group's sequence
};

// block: the workgroup's place among the n_blocks of WAVES waves that walk the list.
template <int NQG, int WAVES>
__device__ __forceinline__ void attn_decode_items(const bf16_t *__restrict__ qkv,
                                                           const int32_t *__restrict__ seq_of_token,
                                                           const int32_t *__restrict__ pos_of_token,
                                                           const int32_t *__restrict__ block_table,
                                                           const bf16_t *__restrict__ k_cache,
                                                           const bf16_t *__restrict__ v_cache,
                                                           bf16_t *__restrict__ out, int ld_out,
                                                           float *__restrict__ part_o, float *__restrict__ part_ml,
                                                           AttnShape sh, const int32_t *__restrict__ plan, int block, int n_blocks) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_items = plan[0] * sh.n_kv;
    const int n_waves = n_blocks * WAVES;
    const int G = sh.n_q / sh.n_kv, TG = 16 / G;
    const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int col_tok = lr / G, col_head = lr % G;   // MFMA column lr of set q = (token q * TG + col_tok, q head col_head)
    const float sscale = 1.4426950408889634f / sqrtf((float)HD);   // log2(e) / sqrt(d)

    // With few rounds the waves that have work are dealt over the workgroups first: what a CU gets from memory is bounded
    // per CU, and four items side by side on one take twice as long as on four (one token behind 2900 positions, 96
    // items: 19.4 -> 9 us; 13 tokens behind 3000, 1248 items: 39 -> 30; 40 behind 2000, 2.5 rounds: 66 -> 63).  From
    // four rounds on all of memory is busy either way, and a chunk's kv heads stay side by side (200 tokens up to 8000
    // positions: 604 us, dealt over the workgroups 608).
    const int gw = n_items < 4 * n_waves ? wave * n_blocks + block : block * WAVES + wave;
    int round = 0;
    auto item_at = [&](int k) { return k * n_waves + ((k & 1) ? n_waves - 1 - gw : gw); };
    int item = item_at(0);
    if (item >= n_items) return;

    auto fetch_item = [&](int it, int &g_out) {
        AttnItem m;
        const int g = it % sh.n_kv, e = it / sh.n_kv;
        const int packed = plan[3 + 2 * e];
        m.c = packed & 0xfffff;
        m.n_tok = packed >> 20;
        m.t = plan[2 + 2 * e];
        m.n_keys = pos_of_token[m.t + m.n_tok - 1] + 1;
        m.seq_pages = (m.n_keys + PS - 1) / PS;
        // A sequence of P pages has ceil(P / chunk_pages) chunks, of equal size up to rounding
        // (ceil(P / chunks) pages, the last one the rest) rather than full ones and a short tail:
        // equal work items are what lets a static deal to the waves finish together.  The sizes
        // depend on the sequence's own length only.
        const int n_chunks = (m.seq_pages + sh.chunk_pages - 1) / sh.chunk_pages;
        const int cp = (m.seq_pages + n_chunks - 1) / n_chunks;
        m.lp_first = m.c * cp;
        const int n_pg = min(cp, m.seq_pages - m.lp_first);
        m.lp_last = m.lp_first + n_pg - 1;
        m.key_end = min(m.n_keys, (m.lp_first + n_pg) * PS);
        m.n_pair = (n_pg + 2 * TILE_PAGES - 1) / (2 * TILE_PAGES);          // a trailing odd tile is walked masked
        m.bt = block_table + (size_t)seq_of_token[m.t] * sh.max_pages_per_seq;
        g_out = g;
        return m;
    };

    u32x4 kreg[2][TILE_PAGES][4];
    u32x2 vreg[2][TILE_PAGES][8];
    bf16x8 qb[NQG][4], qn[NQG][4];
    int nk_cur[NQG], nk_nxt[NQG];                  // keys each column attends (0 for a dead column)

    // tile TL of item M into register buffer B; page indices past the chunk's last page
    // are clamped (their scores are masked, the loads hit L2)
#define DYN_ATTN_LOAD(B, M, GG, TL)                                                                               \
    {                                                                                                             \
        _Pragma("unroll") for (int pi = 0; pi < TILE_PAGES; ++pi) {                                               \
            const int lp = min((M).lp_first + (TL) * TILE_PAGES + pi, (M).lp_last);                               \
            const size_t pg = (size_t)(M).bt[lp] * sh.n_kv + (GG);                                                \
            const bf16_t *kp = k_cache + (pg * PS + lr) * HD + 8 * lq;                                            \
            const bf16_t *vp = v_cache + (pg * HD + lr) * PS + 4 * lq;                                            \
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                                      \
                kreg[B][pi][ks] = *reinterpret_cast<const u32x4 *>(kp + ks * 32);                                 \
            _Pragma("unroll") for (int dt = 0; dt < 8; ++dt)                                                      \
                vreg[B][pi][dt] = *reinterpret_cast<const u32x2 *>(vp + dt * 16 * PS);                            \
        }                                                                                                         \
    }
    // B operands of the score product: column lr of set q = q vector of token t + q*TG + col_tok,
    // head g*G + col_head (zero for columns past the group)
#define DYN_ATTN_LOAD_Q(DST, NK, M, GG)                                                                           \
    _Pragma("unroll") for (int q = 0; q < NQG; ++q) {                                                             \
        const bool live = q * TG + col_tok < (M).n_tok && col_tok < TG;                                           \
        const int tq = (M).t + (live ? q * TG + col_tok : 0);                                                     \
        NK[q] = live ? min(pos_of_token[tq] + 1, (M).key_end) : 0;                                                \
        const bf16_t *qp = qkv + (size_t)tq * ((sh.n_q + 2 * sh.n_kv) * HD) + ((GG) * G + col_head) * HD + 8 * lq; \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {                                                        \
            u32x4 v = *reinterpret_cast<const u32x4 *>(qp + ks * 32);                                             \
            if (!live) v = u32x4{0u, 0u, 0u, 0u};                                                                 \
            DST[q][ks] = __builtin_bit_cast(bf16x8, v);                                                           \
        }                                                                                                         \
    }
#define DYN_ATTN_COMPUTE(B, TL)                                                                                   \
    _Pragma("unroll") for (int q = 0; q < NQG; ++q) {                                                             \
        f32x4 sv[TILE_PAGES];                                                                                     \
        float mx = -INFINITY;                                                                                     \
        _Pragma("unroll") for (int pi = 0; pi < TILE_PAGES; ++pi) {                                               \
            f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};                                                                  \
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                                      \
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[B][pi][ks]),          \
                                                            qb[q][ks], s, 0, 0, 0);                               \
            const int jb = (cur.lp_first + (TL) * TILE_PAGES + pi) * PS + 4 * lq;                                 \
            _Pragma("unroll") for (int r = 0; r < 4; ++r) {                                                       \
                s[r] = (jb + r < nk_cur[q]) ? s[r] * sscale : -INFINITY;                                          \
                mx = fmaxf(mx, s[r]);                                                                             \
            }                                                                                                     \
            sv[pi] = s;                                                                                           \
        }                                                                                                         \
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));                                                                   \
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));                                                                   \
        const float m_new = fmaxf(m_run[q], mx);                                                                  \
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;   /* a column with no key yet stays empty */        \
        const float alpha = __builtin_amdgcn_exp2f(m_run[q] - m_ref);                                             \
        m_run[q] = m_new;                                                                                         \
        l_run[q] *= alpha;                                                                                        \
        _Pragma("unroll") for (int dt = 0; dt < 8; ++dt) acc[q][dt] *= alpha;                                     \
        _Pragma("unroll") for (int pi = 0; pi < TILE_PAGES; ++pi) {                                               \
            f32x4 p;                                                                                              \
            _Pragma("unroll") for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(sv[pi][r] - m_ref);       \
            const bf16x4 pb = __builtin_convertvector(p, bf16x4);                                                 \
            const u32x2 pw = __builtin_bit_cast(u32x2, pb);                                                       \
            l_run[q] += (__uint_as_float(pw[0] << 16) + __uint_as_float(pw[0] & 0xffff0000u)) +                   \
                        (__uint_as_float(pw[1] << 16) + __uint_as_float(pw[1] & 0xffff0000u));                    \
            const int nvalid = cur.key_end - (cur.lp_first + (TL) * TILE_PAGES + pi) * PS - 4 * lq;               \
            _Pragma("unroll") for (int dt = 0; dt < 8; ++dt) {                                                    \
                u32x2 vv = vreg[B][pi][dt];                                                                       \
                if (nvalid < 4) { /* positions past the group's last: keep stale cache bits out of 0 * x */     \
                    vv[0] &= (nvalid > 0 ? 0x0000ffffu : 0u) | (nvalid > 1 ? 0xffff0000u : 0u);                   \
                    vv[1] &= (nvalid > 2 ? 0x0000ffffu : 0u);                                                     \
                }                                                                                                 \
                acc[q][dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vv),             \
                                                                       __builtin_bit_cast(s16x4, pb), acc[q][dt], 0, 0, 0); \
            }                                                                                                     \
        }                                                                                                         \
    }

    int g_cur = 0, g_nxt = 0;
    AttnItem cur = fetch_item(item, g_cur);
    DYN_ATTN_LOAD_Q(qb, nk_cur, cur, g_cur)
    DYN_ATTN_LOAD(0, cur, g_cur, 0)
    while (true) {
        const int next_item = item_at(round + 1);
        const bool more = next_item < n_items;
        // the wave's last pair "prefetches" itself again: harmless loads instead of a conditional branch
        AttnItem nxt = fetch_item(more ? next_item : item, g_nxt);
        f32x4 acc[NQG][8];
        float m_run[NQG], l_run[NQG];
#pragma unroll
        for (int q = 0; q < NQG; ++q) {
            m_run[q] = -INFINITY;
            l_run[q] = 0.f;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) acc[q][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

        for (int pr = 0; pr < cur.n_pair; ++pr) {
            const bool last = pr + 1 == cur.n_pair;
            // buffer 0 holds tile 2 pr (loaded or in flight); scheduling barriers keep each
            // prefetch ahead of the multiply it overlaps
            DYN_ATTN_LOAD(1, cur, g_cur, 2 * pr + 1)
            __builtin_amdgcn_sched_barrier(0);
            DYN_ATTN_COMPUTE(0, 2 * pr)
            __builtin_amdgcn_sched_barrier(0);
            {   // refill buffer 0: this pair's next tile, or tile 0 of the wave's next pair
                const AttnItem src = last ? nxt : cur;
                const int gg = last ? g_nxt : g_cur, tile = last ? 0 : 2 * pr + 2;
                DYN_ATTN_LOAD_Q(qn, nk_nxt, nxt, g_nxt)
                DYN_ATTN_LOAD(0, src, gg, tile)
            }
            __builtin_amdgcn_sched_barrier(0);
            DYN_ATTN_COMPUTE(1, 2 * pr + 1)
            __builtin_amdgcn_sched_barrier(0);
        }

#pragma unroll
        for (int q = 0; q < NQG; ++q) {
            float l = l_run[q];
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
            if (nk_cur[q] > 0 && cur.seq_pages <= sh.chunk_pages) {   // one chunk is all: finished here, the merge leaves the token alone
                const float inv = 1.0f / l;
                bf16_t *y = out + (size_t)(cur.t + q * TG + col_tok) * ld_out + (g_cur * G + col_head) * HD + 4 * lq;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    u32x2 w;
                    w[0] = (uint32_t)f2bf(acc[q][dt][0] * inv) | ((uint32_t)f2bf(acc[q][dt][1] * inv) << 16);
                    w[1] = (uint32_t)f2bf(acc[q][dt][2] * inv) | ((uint32_t)f2bf(acc[q][dt][3] * inv) << 16);
                    *reinterpret_cast<u32x2 *>(y + dt * 16) = w;
                }
            } else if (nk_cur[q] > cur.lp_first * PS) {          // the chunk exists for this column's token
                const size_t pidx = part_index(sh, cur.t + q * TG + col_tok, g_cur * G + col_head, cur.c);
#pragma unroll
                for (int dt = 0; dt < 8; ++dt)
                    *reinterpret_cast<f32x4 *>(part_o + pidx * HD + dt * 16 + 4 * lq) = acc[q][dt];
                if (lq == 0) {
                    part_ml[pidx * 2] = m_run[q];
                    part_ml[pidx * 2 + 1] = l;
                }
            }
        }
        if (!more) break;
        item = next_item;
        ++round;
        cur = nxt;
        g_cur = g_nxt;
#pragma unroll
        for (int q = 0; q < NQG; ++q) {
            nk_cur[q] = nk_nxt[q];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) qb[q][ks] = qn[q][ks];
        }
    }
#undef DYN_ATTN_LOAD
#undef DYN_ATTN_LOAD_Q
#undef DYN_ATTN_COMPUTE
}

template <int NQG>
__global__ __launch_bounds__(256, NQG == 1 ? 2 : 1) void attn_mfma_kernel(const bf16_t *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                           const int32_t *__restrict__ pos_of_token, const int32_t *__restrict__ block_table,
                                                           const bf16_t *__restrict__ k_cache, const bf16_t *__restrict__ v_cache,
                                                           bf16_t *__restrict__ out, int ld_out, float *__restrict__ part_o,
                                                           float *__restrict__ part_ml, AttnShape sh, const int32_t *__restrict__ plan) {
    attn_decode_items<NQG, 4>(qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, plan, blockIdx.x, gridDim.x);
}

// Workgroups of a mixed launch that start on query blocks (mixed_share).  Costs in us of one CU: a position of a decode item 512 bytes at
// 19.5 GB/s, a query block's tile of 64 positions 6 beside decodes; the first, the middle and the last query block stand for all.
__device__ __forceinline__ int mixed_prompt_groups(const int32_t *__restrict__ plan, const int32_t *__restrict__ plan_multi,
                                                   const int32_t *__restrict__ pos_of_token, const int32_t *__restrict__ ct_of_token, const AttnShape &sh,
                                                   int groups) {
    const int entries = plan_multi[0];
    auto tiles = [&](int e) {
        const int t = plan_multi[2 + 2 * e], packed = plan_multi[3 + 2 * e], ct = ct_of_token[t];
        return (min(ct, pos_of_token[t] + (packed >> 20) - (packed & 0xfffff) * ct) + 63) / 64;
    };
    const float prompts = 1.5f * (tiles(0) + 2 * tiles(entries / 2) + tiles(entries - 1)) * entries, decodes = 0.026f * PS * sh.chunk_pages * plan[0];
    return mixed_share(entries * sh.n_kv, prompts, decodes, groups);
}

// Decodes and prompts of one dispatch in one launch, a workgroup per CU: the first (an equal share of every XCD's) claim query blocks, the others
// walk the decode list and then claim query blocks too.  Decodes wait for memory and prompts for the matrix cores: one behind the
// other, each leaves what the other needs idle.  Two launches -> one: 2048 prompt tokens + 64 decodes behind 2048 positions 117 + 67 -> 151 us; steps
// of 60 + 30, 512 + 64, 1000 + 128 and 2500 + 100 tokens 198 / 542 / 858 / 1487 -> 186 / 521 / 821 / 1444 us, 4096 + 64 2052 -> 2056.
__global__ __launch_bounds__(prefill::kWaves * 64, 1) void attn_mixed_kernel(const bf16_t *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                           const int32_t *__restrict__ pos_of_token, const int32_t *__restrict__ block_table,
                                                           const bf16_t *__restrict__ k_cache, const bf16_t *__restrict__ v_cache,
                                                           bf16_t *__restrict__ out, int ld_out, float *__restrict__ part_o,
                                                           float *__restrict__ part_ml, AttnShape sh, const int32_t *__restrict__ plan,
                                                           const int32_t *__restrict__ plan_multi, int32_t *__restrict__ counter,
                                                           const int32_t *__restrict__ ct_of_token) {
    const int prompts = mixed_prompt_groups(plan, plan_multi, pos_of_token, ct_of_token, sh, gridDim.x);
    if ((int)blockIdx.x >= prompts)
        attn_decode_items<1, prefill::kWaves>(qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, plan,
                                              (int)blockIdx.x - prompts, (int)gridDim.x - prompts);
    prefill::attn_prefill_items(qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, plan_multi, counter,
                                ct_of_token);
}

hipError_t launch_attention_generic(int dtype, const void *qkv, const int32_t *seq_of_token,
                                    const int32_t *pos_of_token, const int32_t *block_table, const void *k_cache,
                                    const void *v_cache, void *out, int ld_out, float *part_o, float *part_ml,
                                    const AttnShape &sh, int rows, hipStream_t s, hipEvent_t mid);

bool attention_mfma_supported(int dtype, const AttnShape &sh) {
    return dtype == 1 && sh.head_dim == HD && sh.page_size == PS && sh.n_q % sh.n_kv == 0 && sh.n_q / sh.n_kv <= 16;
}

hipError_t launch_attention(int dtype, const void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                            const int32_t *block_table, const void *k_cache, const void *v_cache, void *out, int ld_out,
                            float *part_o, float *part_ml, int32_t *plan, bool any_single, bool any_multi, const AttnShape &sh, int rows,
                            hipStream_t s, hipEvent_t mid, hipEvent_t pre, bool plan_ready) {
    if (rows <= 0) return hipSuccess;
    if (!attention_mfma_supported(dtype, sh))
        return launch_attention_generic(dtype, qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out,
                                        part_o, part_ml, sh, rows, s, mid);
    // two work lists per dispatch: single-token sequences, multi-token sequences.  They depend on the rows'
    // sequences and positions only: the first layer of a forward builds them, the others walk them again.
    const AttnPlan lists = attn_plan_lists(plan, sh, rows);
    hipError_t e = plan_ready ? hipSuccess : launch_attn_plan(seq_of_token, pos_of_token, plan, sh, rows, s);
    if (e == hipSuccess && pre) e = hipEventRecord(pre, s);
    if (e != hipSuccess) return e;
    const long max_items = (long)rows * sh.n_kv * sh.max_chunks;
    // every workgroup of a persistent launch has to be resident at once (the work is dealt out by
    // wave index): two per CU of the partition the stream runs on
    const int groups = sh.n_cus > 0 && 2 * sh.n_cus < kPersistentGroups ? 2 * sh.n_cus : kPersistentGroups;
    const int grid = (int)std::min<long>(max_items, groups);        // a workgroup per item while they are few
    if (any_single && any_multi) {
        static bool attr_set = false;
        if (!attr_set) {
            e = hipFuncSetAttribute((const void *)attn_mixed_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, prefill::lds_bytes());
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(attn_mixed_kernel, dim3(groups / 2), dim3(prefill::kWaves * 64), prefill::lds_bytes(), s, (const bf16_t *)qkv, seq_of_token, pos_of_token,
                           block_table, (const bf16_t *)k_cache, (const bf16_t *)v_cache, (bf16_t *)out, ld_out, part_o, part_ml, sh, lists.single, lists.multi,
                           lists.multi + 1, lists.ct_of_token);
        e = hipGetLastError();
    } else if (any_single) {
        hipLaunchKernelGGL(attn_mfma_kernel<1>, dim3(grid), dim3(256), 0, s, (const bf16_t *)qkv, seq_of_token,
                           pos_of_token, block_table, (const bf16_t *)k_cache, (const bf16_t *)v_cache, (bf16_t *)out, ld_out, part_o,
                           part_ml, sh, lists.single);
        e = hipGetLastError();
    } else if (any_multi) {
        e = launch_attention_prefill(qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh,
                                     lists.multi, lists.ct_of_token, max_items, groups, s);
    }
    if (e == hipSuccess && mid) e = hipEventRecord(mid, s);
    if (e != hipSuccess) return e;
    return launch_attention_combine(dtype, true, part_o, part_ml, pos_of_token, lists.ct_of_token, out, ld_out, sh, rows, s, lists.multi + 1, true);
}

}  // namespace dyn
