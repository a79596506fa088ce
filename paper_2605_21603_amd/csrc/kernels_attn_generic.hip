// Paged causal attention for what the bf16, 128-wide, 16-position-page kernels do not take (fp32
// storage, other head dims and page sizes), and the split-KV combine step shared by all attention
// kernels.
//
// A token attends cached positions 0..pos of its sequence.  The key range is cut into
// chunks of a fixed number of pages; a chunk gives an un-normalised partial (running max m, sum l,
// weighted values o) per (token, q head).  The combine kernel merges a token's partials in chunk
// order.  Chunk size is a constant of the layer, so the arithmetic a row sees does not depend on
// the batch around it.
//
// attn_tile_kernel is the matrix-core form, for head dims 32..256 and pages of a multiple of 16
// positions; attn_generic_kernel (one wave per (token, q head, chunk), plain loops) takes the rest.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace dyn {

constexpr int kMaxChunkTokens = 512;

// A 256-thread workgroup serves one (query group, kv head, chunk): the tokens of one sequence whose
// positions share an aligned block of 4 * (16 / G) (G = q heads per kv head), all q heads of the kv
// head at once, so a key is fetched once per group instead of once per (token, q head).  The products are
//   S[16 pos, 16 cols]  = K_tile Q^T    (fp32 storage: 16x16x4 fp32 MFMA; bf16: 16x16x32 bf16 MFMA)
//   O^T[d, 16 cols]    += V_tile^T P    (fp32 storage: 16x16x4 fp32 MFMA; bf16: three 16x16x16 bf16 MFMAs)
// with a column per (token, q head).  Scores, probabilities and sums keep 24 bits throughout: beside bf16 values a
// probability goes in as the three bf16 numbers it is the sum of.  The D layout of the first product (lane: column l % 16,
// positions 4 (l / 16) + r) is the B layout of the second (fp32: if its r-th product takes position 4 (l / 16) + r
// as its k index l / 16), and a lane's V operand is then four consecutive positions of one head-dim row.
// A group of one token (decode) gives each of the four waves a quarter of the chunk's positions and
// merges the four in wave order through LDS (without the quarters a decode chunk takes half as long again); a
// group of several tokens gives each wave its own set of 16 columns, and the waves walk the same
// positions (quarters there: a 300-token prompt + 40 decodes 67 against 51 us).  Which
// of the two a token is part of depends on its sequence only, never on the schedule.
// What bounds it is latency - rows, then block table, then pages - and the instructions around a chunk's few tiles
// (with every page in L2 40 decodes of 64-wide heads take 34.6 of 35.5 us), so everything that does not wait for one
// of these is loaded beside it, two tiles of 16 * TP positions are in flight per wave, the block table is
// read with scalar loads a tile ahead (a vector load of a page id waits for every page load issued before it), and
// nothing is divided (TileRule).  The items that exist are a fraction of the (chunk, kv head, token) grid over the
// block table's width - one in twelve for a prompt beside decodes - and a workgroup without one still takes a place and two
// loads' latency, so from 512 workgroups on they are counted in the kernel and dealt out (TileList).  The operator under events,
// dense grid -> dealt out -> without divisions, in the exp2 domain -> V by bf16 products: bf16, 64-wide heads, 300-token
// prompt + 40 decodes at 64..2048 55 -> 37.5 -> 35 -> 32.7 us, 40 decodes alone 35.5 -> 35 -> 33 -> 30.3; bf16, 128-wide,
// 32-position pages, 13 decodes at 200..3000 43 -> 35 -> 33.4 -> 32.7, at 3000 each (no empty workgroups) 47.3 -> 50.8 -> 49.2
// -> 47.1; fp32, 64-wide, 201-token prompt + 24 decodes 31.4 -> 25.6 -> 25.1.
// Four consecutive outputs, rounded to the storage type.
__device__ __forceinline__ void store4(float *y, f32x4 v) { *reinterpret_cast<f32x4 *>(y) = v; }
__device__ __forceinline__ void store4(bf16_t *y, f32x4 v) {
    u32x2 w;
    w[0] = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
    w[1] = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
    *reinterpret_cast<u32x2 *>(y) = w;
}

// Sizes that every item divides by, with their reciprocals (a division is some 35 vector instructions, and with ten of them
// per item an item was more arithmetic around its keys than on them).
struct TileRule {
    double per_block, per_chunk, per_kv;
    int G, TG, block, chunk, g_mul;                                // q heads per kv head, tokens per set of columns, positions per block and per chunk
};
// a / b for 0 <= a < 2^31 and per_b = 1 / b: a + 1/2 is at least 1 / (2 b) away from a multiple of b, the product's error below a / b 2^-51.
__device__ __forceinline__ int quotient(int a, double per_b) { return (int)(((double)a + 0.5) * per_b); }

// What a workgroup serves: a query group's last token row, its chunk and kv head.
struct TileItem { int t_last, c, g, seq, pos, row_seq, row_pos; };   // + that row's sequence and position; lane l's: the l-th row before it

// The n-th of the items that exist, in token order (a group's chunks in a row, kv heads fastest), for up to kListRows
// rows: every thread counts the chunks of the groups that end in its kListRows / 256 rows.
constexpr int kListRows = 1024, kRowsPerThread = kListRows / 256;
struct TileList {
    int upto[kRowsPerThread], before, total;                       // chunks up to and with each of the thread's rows, before its first, of all rows

    __device__ __forceinline__ void build(const int32_t *__restrict__ seq_of_token, const int32_t *__restrict__ pos_of_token, int rows,
                                          const TileRule &rule, int *scratch) {
        const int r0 = threadIdx.x * kRowsPerThread;
        int seq[kRowsPerThread + 1], pos[kRowsPerThread + 1];
#pragma unroll
        for (int i = 0; i <= kRowsPerThread; ++i) {
            const int r = min(r0 + i, rows - 1);
            seq[i] = seq_of_token[r];
            pos[i] = pos_of_token[r];
        }
        int n = 0;
#pragma unroll
        for (int i = 0; i < kRowsPerThread; ++i) {
            const bool ends = r0 + i + 1 >= rows || seq[i + 1] != seq[i] || quotient(pos[i + 1], rule.per_block) != quotient(pos[i], rule.per_block);
            if (r0 + i < rows && ends) n += quotient(pos[i], rule.per_chunk) + 1;
            upto[i] = n;
        }
        int incl = n;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int x = __shfl_up(incl, off, 64);
            if ((int)(threadIdx.x & 63) >= off) incl += x;
        }
        if ((threadIdx.x & 63) == 63) scratch[threadIdx.x >> 6] = incl;
        __syncthreads();
        before = incl - n;
        total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < (int)(threadIdx.x >> 6)) before += scratch[w];
            total += scratch[w];
        }
    }
    // The thread that counted item n says which it is; every thread of the workgroup calls this.
    // `scratch`: two words that the previous call did not use.
    __device__ __forceinline__ void find(int n, int n_kv, const TileRule &rule, int *scratch, int &t_last, int &c, int &g) const {
        const int entry = quotient(n, rule.per_kv), mine = entry - before;
        if (mine >= 0 && mine < upto[kRowsPerThread - 1]) {
            int i = 0, base = 0;
#pragma unroll
            for (int k = 0; k + 1 < kRowsPerThread; ++k)
                if (mine >= upto[k]) { i = k + 1; base = upto[k]; }
            scratch[0] = threadIdx.x * kRowsPerThread + i;
            scratch[1] = mine - base;
        }
        __syncthreads();
        t_last = __builtin_amdgcn_readfirstlane(scratch[0]);
        c = __builtin_amdgcn_readfirstlane(scratch[1]);
        g = n - entry * n_kv;
    }
};

template <typename T, int HD, int TP>
__device__ __forceinline__ void attn_tile(const T *__restrict__ qkv, const int32_t *__restrict__ block_table, const T *__restrict__ k_cache,
                                          const T *__restrict__ v_cache, T *__restrict__ out, int ld_out, float *__restrict__ part_o,
                                          float *__restrict__ part_ml, const AttnShape &sh, const TileRule &rule, const TileItem &item,
                                          float (*merge_o)[16][(HD < 128 ? HD : 128) + 4], float (*merge_ml)[16][2]) {
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int NK = F32 ? HD / 16 : HD / 32, ND = HD / 16;      // 16-byte K operands and 16-row V operands of a lane
    constexpr int MD = HD < 128 ? HD : 128;                        // head-dim indices merged per round
    typedef typename std::conditional<F32, f32x4, u32x2>::type vload_t;   // four positions of V
    const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = item.g, c = item.c;
    const int G = rule.G, TG = rule.TG, tg = rule.block;           // tokens per set of columns, per group
    const int col_tok = (lr * rule.g_mul) >> 16, col_head = lr - col_tok * G;   // this lane's column: a token of the wave's set and a q head
    const int s = item.seq, p_last = item.pos, row_seq = item.row_seq, row_pos = item.row_pos;
    const int n_tok = __popcll(__ballot(lane < tg && lane <= item.t_last && row_seq == s && quotient(row_pos, rule.per_block) == quotient(p_last, rule.per_block)));
    const int t = item.t_last - n_tok + 1, n_keys = p_last + 1;    // the group's first token; keys its last token attends
    const int ps = sh.page_size, ct = rule.chunk, j0 = c * ct;
    const int j1 = min(j0 + ct, n_keys);
    const bool single = n_tok == 1;
    const int32_t *bt = block_table + (size_t)s * sh.max_pages_per_seq;
    const float tiles_per_page = 16.0f / (float)ps;

    const int set0 = single ? 0 : wave * TG;                       // first token of the wave's columns
    const bool live = col_tok < TG && set0 + col_tok < n_tok;
    const int col_pos = __shfl(row_pos, max(n_tok - 1 - set0 - min(col_tok, TG - 1), 0), 64);   // every lane takes part
    const int col_keys = live ? col_pos + 1 : 0;                   // keys the column attends
    u32x4 qf[NK];
    const T *qp = qkv + (size_t)(t + (live ? set0 + col_tok : 0)) * ((sh.n_q + 2 * sh.n_kv) * HD) + (size_t)(g * G + (live ? col_head : 0)) * HD;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        qf[k] = *reinterpret_cast<const u32x4 *>(qp + (F32 ? k * 16 + 4 * lq : k * 32 + 8 * lq));
        if (!live) qf[k] = u32x4{0u, 0u, 0u, 0u};
    }
    // Scores in the exp2 domain where storage is bf16 (the running maximum of a partial too: the merge is told), in the natural one in fp32.
    const float scale = (F32 ? 1.0f : 1.4426950408889634f) / sqrtf((float)HD);
    auto exp_of = [](float x) { return F32 ? expf(x) : __builtin_amdgcn_exp2f(x); };

    // positions this wave walks, [w0, w1), in tiles of 16 * TP from w0 (a multiple of 16), and where live columns
    // begin to differ in what they see
    int w0 = j0, w1 = j1, free_keys = j1;
    if (single) {
        const int n_tile = (j1 - j0 + 16 * TP - 1) / (16 * TP), per = (n_tile + 3) / 4;
        w0 = j0 + min(wave * per, n_tile) * 16 * TP;
        free_keys = w1 = min(j1, w0 + per * 16 * TP);
    } else {
        const int last = __builtin_amdgcn_readlane(row_pos, n_tok - min(set0 + TG, n_tok)), first = __builtin_amdgcn_readlane(row_pos, max(n_tok - 1 - set0, 0));
        w1 = set0 < n_tok ? min(j1, last + 1) : j0;
        free_keys = min(w1, first + 1);
    }
    const int nk = min(col_keys, w1);                              // end of the column's keys in [w0, w1)

    constexpr int NBUF = HD * sizeof(T) > 512 ? 1 : 2;             // register buffers: fp32 256-wide operands fit once
    u32x4 kr[NBUF][TP][NK];
    vload_t vr[NBUF][TP][ND];
    // Sub-tile i of the tile at position j: its 16 positions lie in one page.  Sub-tiles past the end are the last one again.
    auto place = [&](int j, int i, int &slot) {
        const int at = min(j + 16 * i, (w1 - 1) & ~15);
        const int lp = __builtin_amdgcn_readfirstlane((int)(((float)(at >> 4) + 0.5f) * tiles_per_page));   // at / ps, exact below 2^22 tiles
        slot = at - lp * ps;
        return lp;
    };
    int page[TP];                                                  // pages of the tile that is loaded next
    auto look_up = [&](int j) {
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            int slot;
            page[i] = bt[place(j, i, slot)];
        }
    };
    auto load = [&](auto buf, int j) {
        constexpr int B = decltype(buf)::value;
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            int slot;
            place(j, i, slot);
            const size_t pg = (size_t)page[i] * sh.n_kv + g;
            const T *kp = k_cache + (pg * ps + slot + lr) * HD + (F32 ? 4 : 8) * lq;
            const T *vp = v_cache + (pg * HD + lr) * ps + slot + 4 * lq;
#pragma unroll
            for (int k = 0; k < NK; ++k) kr[B][i][k] = *reinterpret_cast<const u32x4 *>(kp + k * (F32 ? 16 : 32));
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) vr[B][i][dt] = *reinterpret_cast<const vload_t *>(vp + (size_t)dt * 16 * ps);
        }
        look_up(j + 16 * TP);
    };
    f32x4 acc[ND];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    auto multiply = [&](auto buf, int j) {
        constexpr int B = decltype(buf)::value;
        // Some live column must not see all of the tile's positions, or the chunk ends in it (wave-uniform):
        // only then are scores and values masked.
        const bool edge = j + 16 * TP > free_keys;
        f32x4 sv[TP];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kr[B][i][k][e]), __uint_as_float(qf[k][e]), a, 0, 0, 0);
                } else {
                    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[B][i][k]), __builtin_bit_cast(bf16x8, qf[k]), a, 0, 0, 0);
                }
            }
            sv[i] = a * scale;
        }
        if (edge) {
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j + 16 * i + 4 * lq + r >= nk) sv[i][r] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < TP; ++i) mx = fmaxf(mx, fmaxf(fmaxf(sv[i][0], sv[i][1]), fmaxf(sv[i][2], sv[i][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx), m_ref = m_new == -INFINITY ? 0.f : m_new;   // a column with no key yet stays empty
        const float alpha = exp_of(m_run - m_ref);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) acc[dt] *= alpha;
        f32x4 p[TP];
#pragma unroll
        for (int i = 0; i < TP; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) p[i][r] = exp_of(sv[i][r] - m_ref);
            l_run += (p[i][0] + p[i][1]) + (p[i][2] + p[i][3]);
        }
        // Edge tiles.  Positions past the group's last key hold stale cache bits, which must not meet their zero
        // probabilities (0 * NaN).  A later token of the group may hold infinities or NaN of its own: as columns
        // differ in what they see, such values are added position by position.
        bool odd[TP];
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            odd[i] = false;
            if (edge) {
                const int nvalid = w1 - (j + 16 * i + 4 * lq);
#pragma unroll
                for (int dt = 0; dt < ND; ++dt) {
                    if constexpr (F32) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            vr[B][i][dt][r] = r < nvalid ? vr[B][i][dt][r] : 0.f;
                            odd[i] |= !(fabsf(vr[B][i][dt][r]) < INFINITY);
                        }
                    } else {
                        u32x2 &v = vr[B][i][dt];
                        v[0] &= (nvalid > 0 ? 0x0000ffffu : 0u) | (nvalid > 1 ? 0xffff0000u : 0u);
                        v[1] &= (nvalid > 2 ? 0x0000ffffu : 0u) | (nvalid > 3 ? 0xffff0000u : 0u);
#pragma unroll
                        for (int h = 0; h < 2; ++h) odd[i] |= (v[h] & 0x7f800000u) == 0x7f800000u || (v[h] & 0x7f80u) == 0x7f80u;
                    }
                }
                odd[i] = __any(odd[i]);
            }
        }
        auto by_position = [&](auto sub) {
            constexpr int i = decltype(sub)::value;
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v;
                    if constexpr (F32) v = vr[B][i][dt][r];
                    else v = __uint_as_float(r & 1 ? vr[B][i][dt][r >> 1] & 0xffff0000u : vr[B][i][dt][r >> 1] << 16);
#pragma unroll 1
                    for (int q = 0; q < 4; ++q) {          // a loop: this is rare, and code in the way costs instruction fetches
                        const f32x4 one = __builtin_amdgcn_mfma_f32_16x16x4f32(lq == q ? v : 0.f, p[i][r], acc[dt], 0, 0, 0);
                        if (j + 16 * i + 4 * q + r < nk) acc[dt] = one;
                    }
                }
        };
        if constexpr (F32) {
            static_for<0, TP>([&](auto sub) {
                constexpr int i = decltype(sub)::value;
                if (odd[i]) { by_position(sub); return; }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int dt = 0; dt < ND; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[B][i][dt][r], p[i][r], acc[dt], 0, 0, 0);
            });
        } else {
            // A probability is the sum of three bf16 numbers, exactly (8 bits of its 24 each, by truncation), and its
            // products with a bf16 value are exact: three bf16 products stand for one in fp32 at 48 cycles instead of 128.
            // (An infinite value gives NaN where a part is zero; the layer's output row is NaN behind either.)
            u32x2 part[3][TP];
#pragma unroll
            for (int i = 0; i < TP; ++i) {
                uint32_t w[3][4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    w[0][r] = __float_as_uint(p[i][r]) & 0xffff0000u;
                    const float rest = p[i][r] - __uint_as_float(w[0][r]);
                    w[1][r] = __float_as_uint(rest) & 0xffff0000u;
                    w[2][r] = __float_as_uint(rest - __uint_as_float(w[1][r]));
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    part[k][i][0] = (w[k][0] >> 16) | (w[k][1] & 0xffff0000u);
                    part[k][i][1] = (w[k][2] >> 16) | (w[k][3] & 0xffff0000u);
                }
            }
            bool any_odd = false;
#pragma unroll
            for (int i = 0; i < TP; ++i) any_odd |= odd[i];
            if (any_odd) {
                static_for<0, TP>([&](auto sub) { by_position(sub); });
            } else {
                static_for<0, TP>([&](auto sub) {
                    constexpr int i = decltype(sub)::value;
#pragma unroll
                    for (int k = 2; k >= 0; --k)
#pragma unroll
                        for (int dt = 0; dt < ND; ++dt)
                            acc[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vr[B][i][dt]), __builtin_bit_cast(s16x4, part[k][i]), acc[dt], 0, 0, 0);
                });
            }
        }
    };
    const std::integral_constant<int, 0> b0;
    const std::integral_constant<int, NBUF - 1> b1;
    if (w0 < w1) {
        look_up(w0);
        if constexpr (NBUF == 1) {
            for (int j = w0; j < w1; j += 16 * TP) {
                load(b0, j);
                multiply(b0, j);
            }
        } else {
            load(b0, w0);
            for (int j = w0; j < w1; j += 32 * TP) {
                load(b1, j + 16 * TP);                             // past the end: the last sub-tile again
                __builtin_amdgcn_sched_barrier(0);
                multiply(b0, j);
                __builtin_amdgcn_sched_barrier(0);
                load(b0, j + 32 * TP);
                __builtin_amdgcn_sched_barrier(0);
                if (j + 16 * TP < w1) multiply(b1, j + 16 * TP);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);

    if (!single) {                                                 // the wave's own columns are complete
        const ColumnEnd end = column_end(col_keys, j0, ct);
        if (end == COLUMN_NOT_MINE) return;
        const int tq = t + set0 + col_tok, h = g * G + col_head;
        if (end == COLUMN_DONE) {
            const float inv = 1.0f / l_run;
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) store4(out + (size_t)tq * ld_out + h * HD + dt * 16 + 4 * lq, acc[dt] * inv);
        } else {
            const size_t pidx = part_index(sh, tq, h, c);
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) *reinterpret_cast<f32x4 *>(part_o + pidx * HD + dt * 16 + 4 * lq) = acc[dt];
            if (lq == 0) { part_ml[pidx * 2] = m_run; part_ml[pidx * 2 + 1] = l_run; }
        }
        return;
    }
    // single token: merge of the four waves, in wave order; a token whose keys fit one chunk is finished here (attn_combine_kernel leaves it alone)
    if (lq == 0) { merge_ml[wave][lr][0] = m_run; merge_ml[wave][lr][1] = l_run; }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, merge_ml[w][lr][0]);
    const float mine = exp_of(m_run - (M == -INFINITY ? 0.f : M));
    for (int round = 0; round < HD / MD; ++round) {
        if (round) __syncthreads();
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
            if (dt / (MD / 16) == round) *reinterpret_cast<f32x4 *>(&merge_o[wave][lr][(dt % (MD / 16)) * 16 + 4 * lq]) = acc[dt] * mine;
        if (round == 0 && lq == 0) merge_ml[wave][lr][1] = l_run * mine;
        __syncthreads();
        for (int u = threadIdx.x; u < G * (MD / 4); u += 256) {
            const int col = u / (MD / 4), i = (u % (MD / 4)) * 4, h = g * G + col;
            f32x4 o = *reinterpret_cast<const f32x4 *>(&merge_o[0][col][i]);
            float L = merge_ml[0][col][1];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(&merge_o[w][col][i]);
                o[0] += x[0]; o[1] += x[1]; o[2] += x[2]; o[3] += x[3];
                L += merge_ml[w][col][1];
            }
            const int d = round * MD + i;
            if (n_keys <= ct) {
                store4(out + (size_t)t * ld_out + h * HD + d, o * (1.0f / L));
            } else {
                const size_t pidx = part_index(sh, t, h, c);
                *reinterpret_cast<f32x4 *>(part_o + pidx * HD + d) = o;
                if (d == 0) {
                    float Mh = -INFINITY;
#pragma unroll
                    for (int w = 0; w < 4; ++w) Mh = fmaxf(Mh, merge_ml[w][col][0]);
                    part_ml[pidx * 2] = Mh;
                    part_ml[pidx * 2 + 1] = L;
                }
            }
        }
    }
}

// LIST: the workgroups walk the items that exist, dealt in turn; else one workgroup per (chunk, kv head, token) of the
// dense grid, of which only a group's last token and the chunks it reaches have work.
template <typename T, int HD, int TP, bool LIST>
__global__ __launch_bounds__(256, HD * sizeof(T) <= 256 ? 2 : 1) void attn_tile_kernel(const T *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                        const int32_t *__restrict__ pos_of_token,
                                                        const int32_t *__restrict__ block_table, const T *__restrict__ k_cache,
                                                        const T *__restrict__ v_cache, T *__restrict__ out, int ld_out,
                                                        float *__restrict__ part_o, float *__restrict__ part_ml, AttnShape sh,
                                                        TileRule rule, int rows, int y0, int y1) {
    __shared__ float merge_o[4][16][(HD < 128 ? HD : 128) + 4];
    __shared__ float merge_ml[4][16][2];
    auto item_of = [&](int t_last, int c, int g) {
        const int row = max(t_last - (int)(threadIdx.x & 63), 0);
        return TileItem{t_last, c, g, seq_of_token[t_last], pos_of_token[t_last], seq_of_token[row], pos_of_token[row]};
    };
    auto serve = [&](const TileItem &item) {
        attn_tile<T, HD, TP>(qkv, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, rule, item, merge_o, merge_ml);
    };
    if constexpr (LIST) {
        __shared__ int scratch[8];
        TileList list;
        list.build(seq_of_token, pos_of_token, rows, rule, scratch);
        const int n_items = list.total * sh.n_kv;
        int n = blockIdx.x, t_last, c, g, turn = 0;
        if (n >= n_items) return;
        auto next = [&]() {                                        // item n; its rows' loads are in flight while the one before is served
            turn ^= 2;
            list.find(n, sh.n_kv, rule, scratch + 4 + turn, t_last, c, g);
            return item_of(t_last, c, g);
        };
        TileItem cur = next();
        while (true) {
            n += gridDim.x;
            const bool more = n < n_items;
            TileItem nxt = cur;
            if (more) nxt = next();
            serve(cur);
            if (!more) break;
            __syncthreads();                                       // the merge arrays are free again
            cur = nxt;
        }
    } else {
        // (chunk, kv head, token), tokens fastest.  Few sequences reach the later chunks: workgroup ids, which go to
        // the 8 XCDs in turn, are rotated inside every eight by their higher bits so that the ones with
        // work, however regularly spaced, spread over all XCDs.
        const unsigned wg = (blockIdx.x & ~7u) | ((blockIdx.x + (blockIdx.x >> 3) + (blockIdx.x >> 6)) & 7u);
        const int t = (int)(wg % rows), y = y0 + (int)(wg / rows);     // y: (chunk, kv head) in [y0, y1) of this launch
        const int g = (int)((unsigned)y % (unsigned)sh.n_kv), c = (int)((unsigned)y / (unsigned)sh.n_kv);
        if (y >= y1) return;
        const int after = min(t + 1, rows - 1), s_after = seq_of_token[after], p_after = pos_of_token[after];
        const TileItem item = item_of(t, c, g);
        if (after > t && s_after == item.seq && quotient(p_after, rule.per_block) == quotient(item.pos, rule.per_block)) return;   // not the last token of its group
        if (c * rule.chunk > item.pos) return;
        serve(item);
    }
}

template <typename T>
__global__ __launch_bounds__(64) void attn_generic_kernel(const T *__restrict__ qkv,
                                                          const int32_t *__restrict__ seq_of_token,
                                                          const int32_t *__restrict__ pos_of_token,
                                                          const int32_t *__restrict__ block_table,
                                                          const T *__restrict__ k_cache, const T *__restrict__ v_cache,
                                                          float *__restrict__ part_o, float *__restrict__ part_ml,
                                                          AttnShape sh) {
    const int c = blockIdx.x % sh.max_chunks;
    const int h = (blockIdx.x / sh.max_chunks) % sh.n_q;
    const int t = blockIdx.x / (sh.max_chunks * sh.n_q);
    const int d = sh.head_dim, ps = sh.page_size, ct = sh.chunk_pages * ps;
    const int n_keys = pos_of_token[t] + 1;
    const int j0 = c * ct;
    if (j0 >= n_keys) return;
    const int j1 = min(j0 + ct, n_keys);
    const int g = h / (sh.n_q / sh.n_kv);
    const int lane = threadIdx.x;
    const int32_t *bt = block_table + (size_t)seq_of_token[t] * sh.max_pages_per_seq;

    __shared__ float qs[2 * kMaxHalfDim];
    __shared__ float sc[kMaxChunkTokens];
    const T *q = qkv + (size_t)t * ((sh.n_q + 2 * sh.n_kv) * d) + h * d;
    for (int i = lane; i < d; i += 64) qs[i] = to_f32<T>(q[i]);
    __syncthreads();

    const float scale = 1.0f / sqrtf((float)d);
    const auto score = [&](int j) {
        const T *kr = k_cache + (((size_t)bt[j / ps] * sh.n_kv + g) * ps + j % ps) * d;
        float acc = 0.f;
        for (int i = 0; i < d; ++i) acc += qs[i] * to_f32<T>(kr[i]);
        return acc * scale;
    };
    // A chunk may hold more positions than sc: its first kMaxChunkTokens scores are kept from the maximum's
    // pass, those of later blocks are computed again and their values added to the partial by the lane that wrote it.
    float mx = -INFINITY;
    for (int j = j0 + lane; j < j1; j += 64) {
        const float x = score(j);
        if (j - j0 < kMaxChunkTokens) sc[j - j0] = x;
        mx = fmaxf(mx, x);
    }
    mx = wave_max(mx);
    float sum = 0.f;
    const size_t pidx = part_index(sh, t, h, c);
    for (int b0 = j0; b0 < j1; b0 += kMaxChunkTokens) {
        const int b1 = min(b0 + kMaxChunkTokens, j1);
        if (b0 > j0) __syncthreads();                   // the last block's probabilities have been read
        for (int j = b0 + lane; j < b1; j += 64) {
            const float p = expf((b0 == j0 ? sc[j - b0] : score(j)) - mx);
            sc[j - b0] = p;
            sum += p;
        }
        __syncthreads();
        for (int i = lane; i < d; i += 64) {
            float acc = b0 == j0 ? 0.f : part_o[pidx * d + i];
            for (int j = b0; j < b1; ++j) {
                const T *vr = v_cache + (((size_t)bt[j / ps] * sh.n_kv + g) * d + i) * ps + j % ps;
                acc += sc[j - b0] * to_f32<T>(*vr);
            }
            part_o[pidx * d + i] = acc;
        }
    }
    sum = wave_sum(sum);
    if (lane == 0) {
        part_ml[pidx * 2] = mx;
        part_ml[pidx * 2 + 1] = sum;
    }
}

// 32 lanes per (token, q head), 8 pairs per 256-thread workgroup; a lane owns 4 consecutive
// head-dim indices.  Partials are merged in chunk order: M = max m_c,
// out = sum_c e(m_c - M) o_c / sum_c e(m_c - M) l_c, where e is exp or exp2 according to the
// domain the producing kernel kept m in.
// A token with more than kMergeSegment chunks (contexts beyond 16384 positions in decode) is
// merged in two levels: first every segment of kMergeSegment chunks into one partial of the same
// (m, l, o) form, stored over the segment's first chunk, then the segments.  Which way a token goes
// depends on its own chunk count only, so its bits do not depend on the batch; the one-level merge
// of a 131072-position context was a 512-step chain on 32 lanes (126 us for one token).
constexpr int kMergeSegment = 64;

template <bool BASE2>
__global__ __launch_bounds__(256) void attn_combine_segments_kernel(float *__restrict__ part_o, float *__restrict__ part_ml,
                                                                    const int32_t *__restrict__ pos_of_token,
                                                                    const int32_t *__restrict__ ct_of_token, AttnShape sh,
                                                                    int n_pairs, int max_segments) {
    const int unit = blockIdx.x * 8 + (threadIdx.x >> 5), sub = threadIdx.x & 31;
    const int pair = unit / max_segments, seg = unit % max_segments;
    if (pair >= n_pairs) return;
    const int t = pair / sh.n_q;
    const int d = sh.head_dim, ct = ct_of_token ? ct_of_token[t] : sh.chunk_pages * sh.page_size;
    const int n_chunks = (pos_of_token[t] + ct) / ct;
    const int c0 = seg * kMergeSegment;
    if (n_chunks <= kMergeSegment || c0 >= n_chunks) return;
    const int n = min(kMergeSegment, n_chunks - c0);
    const size_t next = part_index(sh, 0, 0, 1);           // from a chunk to the one behind it
    const size_t at = part_index(sh, t, pair % sh.n_q, c0);
    float *ml = part_ml + at * 2;
    float *po = part_o + at * d;
    float M = -INFINITY;
    for (int c = sub; c < n; c += 32) M = fmaxf(M, ml[c * next * 2]);
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 32));
    float L = 0.f;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    for (int cb = 0; cb < n; cb += 32) {
        const int c = cb + sub;
        float wgt = 0.f, wl = 0.f;
        if (c < n) {
            const float dm = ml[c * next * 2] - M;
            wgt = BASE2 ? exp2f(dm) : expf(dm);
            wl = wgt * ml[c * next * 2 + 1];
        }
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) wl += __shfl_xor(wl, off, 32);
        L += wl;
        const int nb = min(32, n - cb);
        for (int j0 = 0; j0 < nb; j0 += 4) {
            f32x4 v[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int i = sub * 4 + q * 128;
                    v[j][q] = (j0 + j < nb && i < d) ? *reinterpret_cast<const f32x4 *>(po + (cb + j0 + j) * next * d + i)
                                                      : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float wj = __shfl(wgt, j0 + j, 32);
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[q] += v[j][q] * wj;
            }
        }
    }
    // every lane has read what it needs of the segment (its own four columns of each chunk, and
    // lane 0 the first chunk's (m, l)): the merged partial replaces the segment's first chunk
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = sub * 4 + q * 128;
        if (i < d) *reinterpret_cast<f32x4 *>(po + i) = acc[q];
    }
    if (sub == 0) { ml[0] = M; ml[1] = L; }
}

template <typename T>
__device__ __forceinline__ void merge_store(T *__restrict__ o, const f32x4 &acc, float inv) {
    if constexpr (sizeof(T) == 2) {                    // one 8-byte store (rows and columns are 8-byte aligned)
        u32x2 w;
        w[0] = (uint32_t)f2bf(acc[0] * inv) | ((uint32_t)f2bf(acc[1] * inv) << 16);
        w[1] = (uint32_t)f2bf(acc[2] * inv) | ((uint32_t)f2bf(acc[3] * inv) << 16);
        *reinterpret_cast<u32x2 *>(o) = w;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = from_f32<T>(acc[r] * inv);
    }
}

// Chunks whose partial outputs a half-wave has in flight at once in the final merge (the adds stay in chunk order).
constexpr int kMergeLoads = 8;

// One pair of any number of chunks; `next`: from a partial to the one behind it.
template <typename T, bool BASE2>
__device__ __forceinline__ void merge_pair(const float *__restrict__ ml, const float *__restrict__ po, size_t next, T *__restrict__ out, int n_chunks, int d,
                                           int sub) {
    float M = -INFINITY;
    for (int c = sub; c < n_chunks; c += 32) M = fmaxf(M, ml[c * next * 2]);
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 32));
    // Lane `sub` weighs chunk cb + sub; the weights travel by shuffle so that the value loads
    // of a block of chunks are independent of one another and can all be in flight together.
    float L = 0.f;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};   // head_dim <= 256: two float4 per lane
    for (int cb = 0; cb < n_chunks; cb += 32) {
        const int c = cb + sub;
        float wgt = 0.f, wl = 0.f;
        if (c < n_chunks) {
            const float dm = ml[c * next * 2] - M;
            wgt = BASE2 ? exp2f(dm) : expf(dm);
            wl = wgt * ml[c * next * 2 + 1];
        }
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) wl += __shfl_xor(wl, off, 32);
        L += wl;
        const int nb = min(32, n_chunks - cb);
        for (int j0 = 0; j0 < nb; j0 += kMergeLoads) {
            f32x4 v[kMergeLoads][2];
#pragma unroll
            for (int j = 0; j < kMergeLoads; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int i = sub * 4 + q * 128;
                    v[j][q] = (j0 + j < nb && i < d) ? *reinterpret_cast<const f32x4 *>(po + (cb + j0 + j) * next * d + i)
                                                      : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
            for (int j = 0; j < kMergeLoads; ++j) {
                const float wj = __shfl(wgt, j0 + j, 32);      // 0 beyond the last chunk
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[q] += v[j][q] * wj;
            }
        }
    }
    const float inv = 1.0f / L;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = sub * 4 + q * 128;
        if (i < d) merge_store<T>(out + i, acc[q], inv);
    }
}

// The sum a butterfly over lanes makes of x[0] .. x[N - 1] and zeros (N a power of two).
template <int N>
__device__ __forceinline__ float butterfly_sum(const float (&x)[N]) {
    float v[N];
#pragma unroll
    for (int c = 0; c < N; ++c) v[c] = x[c];
#pragma unroll
    for (int n = N / 2; n >= 1; n >>= 1)
#pragma unroll
        for (int c = 0; c < n; ++c) v[c] += v[c + n];
    return v[0];
}

// U pairs 8 apart of at most N chunks, head_dim at most 128: every load in flight together, each lane weighs all chunks itself.  Same sums in
// the same order as merge_pair.
template <int N, int U, typename T, bool BASE2>
__device__ __forceinline__ void merge_few(const float *__restrict__ ml, const float *__restrict__ po, size_t next, T *__restrict__ out, int n_chunks,
                                          int d, int sub, int live) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const int i = min(sub * 4, d - 4);                     // head_dim is a multiple of 4; lanes past it read the last columns
    f32x2 s[U][N];
    f32x4 v[U][N];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < N; ++c)
            if (c < n_chunks) {
                const size_t at = c * next + (u < live ? u * 8 : 0);
                s[u][c] = *reinterpret_cast<const f32x2 *>(ml + at * 2);
                v[u][c] = *reinterpret_cast<const f32x4 *>(po + at * d + i);
            }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float M = s[u][0][0], wl[N];
#pragma unroll
        for (int c = 1; c < N; ++c)
            if (c < n_chunks) M = fmaxf(M, s[u][c][0]);
        f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < N; ++c) {
            wl[c] = 0.f;
            if (c < n_chunks) {
                const float dm = s[u][c][0] - M, w = BASE2 ? exp2f(dm) : expf(dm);
                wl[c] = w * s[u][c][1];
                acc += v[u][c] * w;
            }
        }
        const float inv = 1.0f / butterfly_sum(wl);
        if (u < live && sub * 4 < d) merge_store<T>(out + u * 8 * d + sub * 4, acc, inv);
    }
}

// Grid: tokens x groups of 8 q heads, a half-wave per (token, head); a token's chunk count is the same for the whole workgroup.  The launch
// is bound by what its waves issue and by the chain of their loads, not by the partials' bytes: where a token has one or two
// chunks, as most tokens of prompts have, its first workgroup merges kMergeHeads groups at a time and the others end at once.  A pair to a
// half-wave, weights by shuffles, chunk counts by a division a thread -> this: 2112 rows 23.1 -> 15.5 us, 4096 prompt tokens of up to two chunks
// 55 -> 28, 128 decodes of up to 16 chunks 8.2 -> 7.4, one token 5.4 -> 4.8, 340 rows of 64-wide heads 6.3 -> 4.8.
constexpr int kMergeHeads = 4;
template <typename T, bool BASE2>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float *__restrict__ part_o,
                                                           const float *__restrict__ part_ml,
                                                           const int32_t *__restrict__ pos_of_token,
                                                           const int32_t *__restrict__ ct_of_token,
                                                           T *__restrict__ out, int ld_out, AttnShape sh,
                                                           int32_t *__restrict__ counter_reset, bool one_chunk_done) {
    // the query-block kernel that ran before this one has drained its work counter: zero it for the
    // next launch that walks the same work list (the next layer of the forward)
    if (counter_reset && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *counter_reset = 0;
    const int t = blockIdx.x, sub = threadIdx.x & 31, d = sh.head_dim;
    const int ct = ct_of_token ? ct_of_token[t] : sh.chunk_pages * sh.page_size;     // per-token chunk size if given
    const int all_chunks = (pos_of_token[t] + ct) / ct;     // ceil((pos + 1) / ct)
    if (one_chunk_done && all_chunks == 1) return;          // the attention kernel wrote this token's output itself
    const size_t chunk = part_index(sh, 0, 0, 1);           // from a chunk to the one behind it
    int h = blockIdx.y * 8 + (threadIdx.x >> 5);
    if (d <= 128 && all_chunks <= 2) {
        if (blockIdx.y) return;
        for (; h < sh.n_q; h += 8 * kMergeHeads) {
            const size_t at = part_index(sh, t, h, 0);
            merge_few<2, kMergeHeads, T, BASE2>(part_ml + at * 2, part_o + at * d, chunk, out + (size_t)t * ld_out + h * d, all_chunks, d, sub,
                                                (sh.n_q - h + 7) / 8);
        }
        return;
    }
    if (h >= sh.n_q) return;
    const size_t at = part_index(sh, t, h, 0);
    const float *const ml = part_ml + at * 2, *const po = part_o + at * d;
    T *const y = out + (size_t)t * ld_out + h * d;
    if (d <= 128 && all_chunks <= 8) {
        merge_few<8, 1, T, BASE2>(ml, po, chunk, y, all_chunks, d, sub, 1);
        return;
    }
    // beyond kMergeSegment chunks the segments kernel has merged every segment into its first chunk
    const int step = all_chunks > kMergeSegment ? kMergeSegment : 1;
    merge_pair<T, BASE2>(ml, po, step * chunk, y, (all_chunks + step - 1) / step, d, sub);
}

// one_chunk_done: the attention kernels finish tokens whose keys fit one chunk themselves.
hipError_t launch_attention_combine(int dtype, bool base2, float *part_o, float *part_ml,
                                    const int32_t *pos_of_token, const int32_t *ct_of_token, void *out, int ld_out,
                                    const AttnShape &sh, int rows, hipStream_t s, int32_t *counter_reset, bool one_chunk_done) {
    if (one_chunk_done && sh.max_chunks == 1 && !counter_reset) return hipSuccess;       // no token has anything to merge
    const int n_pairs = rows * sh.n_q;
    const dim3 block(256);
    if (sh.max_chunks > kMergeSegment) {       // some token may have that many chunks: first level of the merge
        const int max_segments = (sh.max_chunks + kMergeSegment - 1) / kMergeSegment;
        const dim3 seg_grid((unsigned)(((size_t)n_pairs * max_segments + 7) / 8));
        if (base2) hipLaunchKernelGGL(attn_combine_segments_kernel<true>, seg_grid, block, 0, s, part_o, part_ml, pos_of_token, ct_of_token, sh, n_pairs, max_segments);
        else hipLaunchKernelGGL(attn_combine_segments_kernel<false>, seg_grid, block, 0, s, part_o, part_ml, pos_of_token, ct_of_token, sh, n_pairs, max_segments);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#define DYN_COMBINE(T, B2)                                                                                                                              \
    hipLaunchKernelGGL((attn_combine_kernel<T, B2>), dim3(rows, (sh.n_q + 7) / 8), block, 0, s, part_o, part_ml, pos_of_token, ct_of_token, (T *)out, \
                       ld_out, sh, counter_reset, one_chunk_done)
    if (dtype == 0) {
        if (base2) DYN_COMBINE(float, true); else DYN_COMBINE(float, false);
    } else {
        if (base2) DYN_COMBINE(bf16_t, true); else DYN_COMBINE(bf16_t, false);
    }
#undef DYN_COMBINE
    return hipGetLastError();
}

namespace {
// The matrix-core form reads K and q 16 bytes and V four positions at a time.
bool attn_tile_supported(const AttnShape &sh, const void *k_cache, const void *v_cache) {
    const int d = sh.head_dim;
    return (d == 32 || d == 64 || d == 128 || d == 256) && sh.page_size % 16 == 0 && sh.n_q / sh.n_kv <= 16 &&
           (((uintptr_t)k_cache | (uintptr_t)v_cache) & 15) == 0;
}

// A grid's threads along x are counted in 32 bits, and what does not fit wraps without an error: 1024 rows of 32 kv heads
// under a table of 512 chunks are 2^32 threads.  Larger grids go as several launches, each a range of (chunk, kv head), or
// of rows in the general form.
constexpr size_t kTileGrid = (size_t)1 << 23;          // workgroups of a launch of the tile form, about
constexpr size_t kGeneralGrid = (size_t)1 << 25;       // of the general form

// Up to kListGrid workgroups the dense grid is resident at once and its items start a scan earlier (4 tokens behind 128
// positions: 14.8 us either way, one workgroup per CU).  Beyond, as many workgroups as are resident walk the list: two per CU with
// 256-byte rows (at 1024 workgroups 13 decodes of 200..3000 positions 39.8 us, at 512 34.8), else four (300 + 40 tokens: 512 / 768 / 1024 /
// 2048 workgroups 41.6 / 39.1 / 36.9 / 38.2).
constexpr size_t kListGrid = 512;


template <typename T, int HD, int TP>
void launch_attn_tile(hipStream_t s, const void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                      const int32_t *block_table, const void *k_cache, const void *v_cache, void *out, int ld_out, float *part_o,
                      float *part_ml, const AttnShape &sh, int rows) {
    const int n_y = sh.n_kv * sh.max_chunks;
    const size_t dense = (size_t)rows * n_y;
    const int G = sh.n_q / sh.n_kv, block = 4 * (16 / G), chunk = sh.chunk_pages * sh.page_size;
    const TileRule rule{1.0 / block, 1.0 / chunk, 1.0 / sh.n_kv, G, 16 / G, block, chunk, 65536 / G + 1};
#define DYN_TILE_LAUNCH(LIST, GRID, Y0, Y1)                                                                                              \
    hipLaunchKernelGGL((attn_tile_kernel<T, HD, TP, LIST>), dim3(GRID), dim3(256), 0, s, (const T *)qkv, seq_of_token, pos_of_token,     \
                       block_table, (const T *)k_cache, (const T *)v_cache, (T *)out, ld_out, part_o, part_ml, sh, rule, rows, Y0, Y1)
    if (rows <= kListRows && dense > kListGrid) {
        DYN_TILE_LAUNCH(true, (unsigned)std::min<size_t>(dense, HD * sizeof(T) >= 256 ? 512 : 1024), 0, n_y);
        return;
    }
    const int step = (int)std::max<size_t>(kTileGrid / rows, 1);
    for (int y0 = 0; y0 < n_y; y0 += std::min(step, n_y - y0)) {
        const int y1 = y0 + std::min(step, n_y - y0);
        DYN_TILE_LAUNCH(false, (unsigned)(((size_t)rows * (y1 - y0) + 7) / 8 * 8), y0, y1);               // whole eights of workgroups
    }
#undef DYN_TILE_LAUNCH
}
}  // namespace

hipError_t launch_attention_generic(int dtype, const void *qkv, const int32_t *seq_of_token,
                                    const int32_t *pos_of_token, const int32_t *block_table, const void *k_cache,
                                    const void *v_cache, void *out, int ld_out, float *part_o, float *part_ml,
                                    const AttnShape &sh, int rows, hipStream_t s, hipEvent_t mid) {
    if (rows <= 0) return hipSuccess;
    if (rows >= 1 << 24) return hipErrorInvalidConfiguration;
    const bool tile = attn_tile_supported(sh, k_cache, v_cache);
    if (tile) {
        // positions per tile: two sub-tiles of 16 where a lane's K and V operands of both fit beside the
        // accumulators twice over, else one
#define DYN_TILE(T, HD, TP) launch_attn_tile<T, HD, TP>(s, qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, rows)
        if (dtype == 0) {
            switch (sh.head_dim) {
                case 32: DYN_TILE(float, 32, 2); break;
                case 64: DYN_TILE(float, 64, 2); break;
                case 128: DYN_TILE(float, 128, 1); break;
                default: DYN_TILE(float, 256, 1); break;
            }
        } else {
            switch (sh.head_dim) {
                case 32: DYN_TILE(bf16_t, 32, 2); break;
                case 64: DYN_TILE(bf16_t, 64, 2); break;
                case 128: DYN_TILE(bf16_t, 128, 1); break;
                default: DYN_TILE(bf16_t, 256, 1); break;
            }
        }
#undef DYN_TILE
    } else {
        const size_t per_row = (size_t)sh.n_q * sh.max_chunks, width = (size_t)(sh.n_q + 2 * sh.n_kv) * sh.head_dim;
        const int step = (int)std::max<size_t>(kGeneralGrid / per_row, 1);
        if (per_row >= (size_t)1 << 26) return hipErrorInvalidConfiguration;
        for (int r0 = 0; r0 < rows; r0 += std::min(step, rows - r0)) {
            const dim3 grid((unsigned)(std::min(step, rows - r0) * per_row));
            float *const po = part_o + part_index(sh, r0, 0, 0) * sh.head_dim, *const pml = part_ml + part_index(sh, r0, 0, 0) * 2;
            if (dtype == 0)
                hipLaunchKernelGGL(attn_generic_kernel<float>, grid, dim3(64), 0, s, (const float *)qkv + r0 * width, seq_of_token + r0,
                                   pos_of_token + r0, block_table, (const float *)k_cache, (const float *)v_cache, po, pml, sh);
            else
                hipLaunchKernelGGL(attn_generic_kernel<bf16_t>, grid, dim3(64), 0, s, (const bf16_t *)qkv + r0 * width, seq_of_token + r0,
                                   pos_of_token + r0, block_table, (const bf16_t *)k_cache, (const bf16_t *)v_cache, po, pml, sh);
        }
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && mid) e = hipEventRecord(mid, s);
    if (e != hipSuccess) return e;
    return launch_attention_combine(dtype, tile && dtype == 1, part_o, part_ml, pos_of_token, nullptr, out, ld_out, sh, rows, s, nullptr, tile);
}

}  // namespace dyn
