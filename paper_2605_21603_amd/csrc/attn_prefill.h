// Causal paged attention for the tokens of multi-token sequences (prefill chunks): the
// compute-bound form of the layer's attention (the paper's compute-bound operator class,
// Section 2), bf16 caches, head_dim 128, 16-position pages.
//
// An 8-wave workgroup serves one query block - up to 16 * (16 / G) tokens (64 with G = 4 q heads per kv
// head) of one sequence whose positions fall in one aligned block - against one chunk of cached positions (1024, more behind
// a long prefix or for a long prompt: prompt_chunk_positions) of one kv head.  K and V tiles of 64 positions (four pages each, 32 KB together) go from
// global memory straight into an LDS ring with direct loads, once per workgroup, and all eight waves read
// their MFMA operands from there: a key is fetched once per query block and q-head
// group, and the waves hold no K/V staging registers.  A wave owns two sets of 16 columns
// (64 accumulator registers): everything fits the 256 vector registers of a wave at two
// waves per SIMD, so one wave's softmax overlaps another's matrix products and no operand
// ever sits in an accumulation register it has to be copied out of.
//   S[64 pos, 32 cols]  = K_tile[64, 128] Q^T[128, 32]       (32 x mfma 16x16x32 per wave)
//   O^T[128, 32 cols]  += V_tile^T[128, 64] P[64, 32]        (32 x mfma 16x16x32 per wave)
// A column is (token, q head of the kv head's group); the D layout of the first product
// (lane: column l % 16, positions 4 (l / 16) + r of a page) is the B layout of the second
// with the k index running over (one page: 4 positions, the next: 4 positions), and V's
// position-fastest page layout makes the matching A operand two 8-byte LDS reads.
// K rows are 256 bytes, so their 16-byte columns are XOR-swizzled with the row on the way in
// (the direct load's source address is permuted, its LDS destination cannot be).
// The waves work in two groups half a tile apart, one multiplying while the other does its softmax (the
// tile loop says how): in step, with all eight waves in the same part of a tile, the matrix pipes idled
// through every softmax.  Chunk kernel, one sequence: 4096 tokens behind 8192 positions 860 -> 728 us (0.94 PFLOP/s), 1000 behind
// 8192 234 -> 193, 4096 alone 218 -> 204, 2048 alone unchanged (68 us).  What a phase waits for now is neither
// the exponentials (without any softmax 690 us), nor the operand reads (three V groups in flight instead of
// one, other bank swizzles: no change), nor the tile loads (without them 650 us): the two groups' halves
// take about as long as each other, and each the sum of its latencies.
// Online softmax in the exp2 domain; the chunk's partial (m, l, o) goes to the split-KV
// arrays and attn_combine_kernel merges a token's chunks in order.
#pragma once
#include "common.h"
#include "kernels.h"

namespace dyn {

namespace prefill {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int HD = 128, PS = 16;
constexpr int kSets = 2;                      // sets of 16 MFMA columns per wave
constexpr int kWaves = 8;                     // waves per workgroup
constexpr int kTP = 4;                         // pages (16 positions each) per K/V tile
constexpr int kRing = 3, kTile = 2 * kTP * 4096;   // LDS ring of K/V tiles: kTP K pages, then kTP V pages, 4 KB each

// Maximum of three and of two (the operands are never signalling: no canonicalising moves as fmaxf has them).
__device__ __forceinline__ float max3(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48, on the vector ALU (a shuffle goes through LDS).
__device__ __forceinline__ float quad_max(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ void wait_vm(int n) {   // s_waitcnt vmcnt(n) only
    if (n == 4) __builtin_amdgcn_s_waitcnt(0x0f74);
    else __builtin_amdgcn_s_waitcnt(0x0f70);
}

// The items of the multi-token list, claimed until none is left, by a workgroup of kWaves * 64 threads with lds_bytes() of dynamic LDS.
__device__ __forceinline__ void attn_prefill_items(const bf16_t *__restrict__ qkv,
                                                              const int32_t *__restrict__ seq_of_token,
                                                              const int32_t *__restrict__ pos_of_token,
                                                              const int32_t *__restrict__ block_table,
                                                              const bf16_t *__restrict__ k_cache,
                                                              const bf16_t *__restrict__ v_cache,
                                                              bf16_t *__restrict__ out, int ld_out,
                                                              float *__restrict__ part_o, float *__restrict__ part_ml,
                                                              AttnShape sh, const int32_t *__restrict__ plan, int32_t *__restrict__ counter,
                                                              const int32_t *__restrict__ ct_of_token) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int32_t *pid = reinterpret_cast<int32_t *>(lds + kRing * kTile);      // physical pages of the chunk
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int late = wave / (kWaves / 2);                                // group of the wave (see the tile loop); it also copies V instead of K
    const int lr = lane & 15, lq = lane >> 4;
    const int G = sh.n_q / sh.n_kv, TG = 16 / G;                         // tokens per set of 16 columns
    const int col_tok = lr / G, col_head = lr % G;
    const int wave_tok0 = wave * kSets * TG;                             // first token of the block this wave owns
    const float sscale = 1.4426950408889634f / sqrtf((float)HD);
    const int n_items = plan[0] * sh.n_kv;
    const size_t row_elems = (size_t)(sh.n_q + 2 * sh.n_kv) * HD;

    // Work items are claimed from a counter in the list's header (zeroed by the work-list kernel),
    // longest first: the list is in token order, a block's keys grow with its position, so it is
    // walked from the back.  A few hundred claims per launch; which workgroup computes an item
    // does not touch its result.
    int32_t *claim = reinterpret_cast<int32_t *>(lds + kRing * kTile) + kPrefillChunkPagesMax;
    for (;;) {
        __builtin_amdgcn_s_waitcnt(0x0f70);                               // the previous item's stores and trailing tile loads
        __syncthreads();                                                  // everyone has read the previous claim and left the ring
        if (tid == 0) *claim = atomicAdd(counter, 1);
        __syncthreads();
        const int taken = *claim;
        if (taken >= n_items) break;
        const int item = n_items - 1 - taken;
        const int g = item % sh.n_kv, e = item / sh.n_kv;
        const int t0 = plan[2 + 2 * e], packed = plan[3 + 2 * e];
        const int c = packed & 0xfffff, n_tok = packed >> 20;
        const int n_keys = pos_of_token[t0 + n_tok - 1] + 1;             // keys the block's last token attends
        const int seq_pages = (n_keys + PS - 1) / PS;
        const int chunk_pages = ct_of_token[t0] / PS;                     // the same for all tokens of an aligned position block
        const int lp0 = c * chunk_pages;
        const int n_pg = min(chunk_pages, seq_pages - lp0);
        const int n_tile = (n_pg + kTP - 1) / kTP;
        const int32_t *bt = block_table + (size_t)seq_of_token[t0] * sh.max_pages_per_seq;

        if (tid < chunk_pages) pid[tid] = bt[lp0 + min(tid, n_pg - 1)];

        // this wave's columns: B operands of the score product and the keys each column attends
        bf16x8 qb[kSets][4];
        int nk[kSets];
#pragma unroll
        for (int q = 0; q < kSets; ++q) {
            const int ti = wave_tok0 + q * TG + col_tok;
            const bool live = col_tok < TG && ti < n_tok;
            const int tq = t0 + (live ? ti : 0);
            nk[q] = live ? pos_of_token[tq] + 1 : 0;
            const bf16_t *qp = qkv + (size_t)tq * row_elems + (size_t)(g * G + col_head) * HD + 8 * lq;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                u32x4 v = *reinterpret_cast<const u32x4 *>(qp + ks * 32);
                if (!live) v = u32x4{0u, 0u, 0u, 0u};
                qb[q][ks] = __builtin_bit_cast(bf16x8, v);
            }
        }
        // keys the wave's last live token attends (positions are consecutive within the block)
        const int wave_keys = wave_tok0 < n_tok ? pos_of_token[t0 + min(wave_tok0 + kSets * TG, n_tok) - 1] + 1 : 0;
        // keys its first token attends; columns of dead tokens or heads carry zeros and are never stored
        const int wave_min_keys = wave_tok0 < n_tok ? pos_of_token[t0 + wave_tok0] + 1 : 0;
        __syncthreads();                                                  // pid is visible

        // Wave w copies one 4 KB page of every tile: K pages 0..3 (waves 0..3), V pages 0..3 (waves 4..7).
        const int wpage = wave & (kTP - 1);
        auto issue = [&](int tile) {
            const int tcl = min(tile, n_tile - 1);                        // past the end: a harmless reload
            const int pg = pid[min(kTP * tcl + wpage, n_pg - 1)];
            unsigned char *dst = lds + (tile % kRing) * kTile + late * (kTP * 4096) + wpage * 4096;
            const size_t page_elems = ((size_t)pg * sh.n_kv + g) * (PS * HD);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bf16_t *src;
                if (late) {
                    const int r = j * 32 + (lane >> 1), h = lane & 1;     // V row (head-dim index), 16-byte half in LDS
                    src = v_cache + page_elems + r * PS + ((h ^ ((r >> 2) & 1)) << 3);
                } else {
                    const int r = j * 4 + (lane >> 4), cs = lane & 15;    // K row, 16-byte slot in LDS
                    src = k_cache + page_elems + r * HD + ((cs ^ (r & 7)) << 3);
                }
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                                 (__attribute__((address_space(3))) void *)(dst + j * 1024), 16, 0, 0);
            }
        };

        f32x4 acc[kSets][8], acc_l[kSets];   // O^T tiles; row sums of P (every row of acc_l holds the column's denominator)
        float m_run[kSets];                  // the reference maximum the column's exponentials are taken against (scaled, log2 domain)
#pragma unroll
        for (int q = 0; q < kSets; ++q) {
            m_run[q] = -INFINITY;
            acc_l[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) acc[q][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
        // V operand: 8 bytes (4 positions) of a 32-byte row.  The row's 16-byte halves are stored
        // swapped when bit 2 of the row is set, which spreads the 16 rows a read touches over
        // twice as many banks as the plain layout.
        const int v_off = lr * 32 + ((((lq >> 1) ^ (lr >> 2)) & 1) << 4) + ((lq & 1) << 3);

        // Operand reads from the ring are assembly with hand-placed waits (common.h): a V operand group is read
        // while the previous group's value products issue, a page's K operands while the previous page's
        // score products issue.  The K operand of k
        // step ks sits in 16-byte column (4 ks + lq) ^ (lr & 7) of row lr: two lane addresses (bit 2 of
        // the column is ks & 1 flipped by bit 2 of the row) and an immediate of 0 or 128 bytes.
        const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
        const unsigned k_lane0 = lr * 256 + (((lq ^ (lr & 3)) + 4 * ((lr >> 2) & 1)) << 4);
        const unsigned k_lane1 = lr * 256 + (((lq ^ (lr & 3)) + 4 * (((lr >> 2) & 1) ^ 1)) << 4);

        // positions past the block's last key (in the chunk's last tile) hold stale cache bits, which must not
        // meet their zero probabilities (0 * NaN): the wave that copied a V page clears them in LDS
        auto clear_stale = [&](int tile) {
            const int nv = n_keys - (lp0 + kTP * tile + wpage) * PS;     // valid positions of this wave's page
            if (nv >= PS) return;
            unsigned char *pb0 = lds + (tile % kRing) * kTile + kTP * 4096 + wpage * 4096;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = j * 32 + (lane >> 1), h = (lane & 1) ^ ((r >> 2) & 1);   // V row, half of its positions in this slot
                const int n = nv - 8 * h;
                u32x4 *w = reinterpret_cast<u32x4 *>(pb0 + j * 1024 + lane * 16);
                u32x4 x = *w;
#pragma unroll
                for (int d = 0; d < 4; ++d) x[d] &= (n > 2 * d ? 0x0000ffffu : 0u) | (n > 2 * d + 1 ? 0xffff0000u : 0u);
                *w = x;
            }
            wait_lgkmcnt<0>();
        };

        // The eight waves run in two groups half a tile apart: while waves 0..3 (one per SIMD) issue the matrix
        // products of a tile, waves 4..7 do the softmax of theirs, and the other way round, with a barrier
        // between the halves.  In phase 2 i the early group multiplies: V of tile i - 1 by its probabilities,
        // then K of tile i; in phase 2 i + 1 it does tile i's softmax; the late group is one phase behind.  K of a tile
        // is read in phases 2 i and 2 i + 1, its V in 2 i + 2 and 2 i + 3, so at the start of phase 2 i the K slot of
        // tile i - 1 and the V slot of tile i - 2 are free: the early waves issue K of tile i + 2, the late ones V of
        // tile i + 1, and what phase 2 i reads has landed when each wave's loads but the last four have.
        f32x4 sv[kSets][kTP];                                             // raw scores q . k of the tile in flight
        bf16x8 pb[kSets][kTP / 2];                                        // probabilities: one k = 32 operand per pair of pages
        auto visible = [&](int ti) { return (lp0 + kTP * ti) * PS < wave_keys; };   // wave-uniform: some position of the tile is
        // the query operands are in their registers before the first direct load is issued: a wait for them
        // inside the loop would be a wait for the ring
#pragma unroll
        for (int q = 0; q < kSets; ++q)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(qb[q][ks]));
        issue(0);
        if (!late) issue(1);
        if (late) {
            wait_vm(0);
            if (n_tile == 1) clear_stale(0);
        } else {
            wait_vm(4);
        }
        __builtin_amdgcn_s_barrier();                                     // tile 0 is there
        if (late) {
            issue(1);
            __builtin_amdgcn_s_barrier();                                 // phase 0
        }
#pragma clang loop unroll(disable)
        for (int ti = 0; ti <= n_tile; ++ti) {                            // one copy of the body: no peeled first round
            if (!late) issue(ti + 2);
            const unsigned tb = lds0 + (unsigned)(ti % kRing) * kTile, tp = lds0 + (unsigned)((ti + kRing - 1) % kRing) * kTile;
            const unsigned ka0 = tb + k_lane0, ka1 = tb + k_lane1, va = tp + kTP * 4096 + (unsigned)v_off;
            __builtin_amdgcn_s_setprio(1);
            if (ti > 0 && visible(ti - 1)) {
                // V operands of output rows 16 dt .. 16 dt + 15, one 8-byte read per page; group 0 is in flight
                // during the denominator's products
                u32x2 vx[2][kTP];
                auto read_v = [&](u32x2 (&x)[kTP], auto dt_c) {
                    static_for<0, kTP>([&](auto pi_c) {
                        x[decltype(pi_c)::value] = lds_read8<decltype(pi_c)::value * 4096 + decltype(dt_c)::value * 512>(va);
                    });
                };
                read_v(vx[0], std::integral_constant<int, 0>());
                // the denominator sums the probabilities exactly as the value product sees them (rounded
                // to bf16): one more matrix product, against a block of ones
#pragma unroll
                for (int pp = 0; pp < kTP / 2; ++pp)
#pragma unroll
                    for (int q = 0; q < kSets; ++q) acc_l[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[q][pp], acc_l[q], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, 8>([&](auto dt_c) {
                    constexpr int dt = decltype(dt_c)::value;
                    if constexpr (dt + 1 < 8) {
                        read_v(vx[(dt + 1) & 1], std::integral_constant<int, dt + 1>());
                        wait_lgkmcnt<kTP>();                              // group dt has arrived
                    } else {
                        wait_lgkmcnt<0>();
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int pp = 0; pp < kTP / 2; ++pp) {
                        const u32x2 x0 = vx[dt & 1][2 * pp], x1 = vx[dt & 1][2 * pp + 1];
                        const bf16x8 vf = __builtin_bit_cast(bf16x8, u32x4{x0[0], x0[1], x1[0], x1[1]});
#pragma unroll
                        for (int q = 0; q < kSets; ++q)
                            acc[q][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pb[q][pp], acc[q][dt], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            if (ti < n_tile && visible(ti)) {
                auto read_k = [&](bf16x8 (&kf)[4], auto pi) {
                    constexpr int OFF = decltype(pi)::value * 4096;
                    kf[0] = lds_read16<OFF>(ka0);
                    kf[1] = lds_read16<OFF>(ka1);
                    kf[2] = lds_read16<OFF + 128>(ka0);
                    kf[3] = lds_read16<OFF + 128>(ka1);
                };
                bf16x8 kf[2][4];
                read_k(kf[0], std::integral_constant<int, 0>());
                static_for<0, kTP>([&](auto pi_c) {
                    constexpr int pi = decltype(pi_c)::value;
                    if constexpr (pi + 1 < kTP) {
                        read_k(kf[(pi + 1) & 1], std::integral_constant<int, pi + 1>());
                        wait_lgkmcnt<4>();                                // page pi's four operands have arrived
                    } else {
                        wait_lgkmcnt<0>();
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < kSets; ++q) sv[q][pi] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int q = 0; q < kSets; ++q) sv[q][pi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[pi & 1][ks], qb[q][ks], sv[q][pi], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            __builtin_amdgcn_s_setprio(0);
            if (late) {                                                   // V of tile ti is in the ring before the next phase reads it
                wait_vm(4);
                if (ti == n_tile - 1) clear_stale(ti);
            }
            __builtin_amdgcn_s_barrier();
            if (late) issue(ti + 2);
            if (ti < n_tile && visible(ti)) {
                const int key0 = (lp0 + kTP * ti) * PS;
                // Causal mask: only the last tiles of a block have positions that some live column of
                // the wave must not see (wave-uniform test).
                if (key0 + kTP * PS > wave_min_keys) {
#pragma unroll
                    for (int q = 0; q < kSets; ++q)
#pragma unroll
                        for (int pi = 0; pi < kTP; ++pi)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (key0 + pi * PS + 4 * lq + r >= nk[q]) sv[q][pi][r] = -INFINITY;
                }
                // The maxima below are assembly (max3), for whose operands the compiler places no wait states: the products'
                // results are in their registers behind this, wherever it puts the rest (4096 tokens behind 8192 positions: the step takes 2463 us with and without).
                static_assert(kSets == 2 && kTP == 4, "every score tile passes through");
                asm volatile("s_nop 15" : "+v"(sv[0][0]), "+v"(sv[0][1]), "+v"(sv[0][2]), "+v"(sv[0][3]),
                                          "+v"(sv[1][0]), "+v"(sv[1][1]), "+v"(sv[1][2]), "+v"(sv[1][3]));
                bool rescale = false;
                float alpha[kSets];
#pragma unroll
                for (int q = 0; q < kSets; ++q) {
                    float half_mx[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f32x4 x = sv[q][2 * h], y = sv[q][2 * h + 1];
                        half_mx[h] = max3(max3(max3(x[0], x[1], x[2]), x[3], y[0]), max3(y[1], y[2], y[3]), y[0]);
                    }
                    const float mx = quad_max(max3(half_mx[0], half_mx[1], half_mx[1])) * sscale;
                    // The reference maximum follows the true one lazily: it moves only when a score
                    // exceeds it by more than 2^8, so exponentials stay below 256 (exact in what
                    // follows: the final division by the denominator cancels the reference) and the
                    // accumulators are rescaled a few times per block instead of on every tile.
                    const bool move = mx > m_run[q] + 8.0f;
                    const float m_new = move ? mx : m_run[q];
                    const float m_ref = m_new == -INFINITY ? 0.f : m_new;    // a column with no key yet stays empty
                    alpha[q] = move ? __builtin_amdgcn_exp2f(m_run[q] - m_ref) : 1.0f;
                    rescale |= move;
                    m_run[q] = m_new;
#pragma unroll
                    for (int pp = 0; pp < kTP / 2; ++pp) {
                        f32x4 p0, p1;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            p0[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[q][2 * pp][r], sscale, -m_ref));
                            p1[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[q][2 * pp + 1][r], sscale, -m_ref));
                        }
                        const u32x2 w0 = __builtin_bit_cast(u32x2, __builtin_convertvector(p0, bf16x4));
                        const u32x2 w1 = __builtin_bit_cast(u32x2, __builtin_convertvector(p1, bf16x4));
                        pb[q][pp] = __builtin_bit_cast(bf16x8, u32x4{w0[0], w0[1], w1[0], w1[1]});
                    }
                }
                if (__any(rescale)) {
#pragma unroll
                    for (int q = 0; q < kSets; ++q) {
                        acc_l[q] *= alpha[q];
#pragma unroll
                        for (int dt = 0; dt < 8; ++dt) acc[q][dt] *= alpha[q];
                    }
                }
            }
            if (!late) wait_vm(4);                                        // K of tile ti + 1 is in the ring
            __builtin_amdgcn_s_barrier();
        }
        if (!late) __builtin_amdgcn_s_barrier();                          // the late group's last phase

#pragma unroll
        for (int q = 0; q < kSets; ++q) {
            const ColumnEnd end = column_end(nk[q], lp0 * PS, chunk_pages * PS);
            if (end == COLUMN_NOT_MINE) continue;
            if (end == COLUMN_DONE) {
                const float inv = 1.0f / acc_l[q][0];
                bf16_t *y = out + (size_t)(t0 + wave_tok0 + q * TG + col_tok) * ld_out + (g * G + col_head) * HD + 4 * lq;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    u32x2 w;
                    w[0] = (uint32_t)f2bf(acc[q][dt][0] * inv) | ((uint32_t)f2bf(acc[q][dt][1] * inv) << 16);
                    w[1] = (uint32_t)f2bf(acc[q][dt][2] * inv) | ((uint32_t)f2bf(acc[q][dt][3] * inv) << 16);
                    *reinterpret_cast<u32x2 *>(y + dt * 16) = w;
                }
            } else {
                const size_t pidx = part_index(sh, t0 + wave_tok0 + q * TG + col_tok, g * G + col_head, c);
#pragma unroll
                for (int dt = 0; dt < 8; ++dt)
                    *reinterpret_cast<f32x4 *>(part_o + pidx * HD + dt * 16 + 4 * lq) = acc[q][dt];
                if (lq == 0) {
                    part_ml[pidx * 2] = m_run[q];
                    part_ml[pidx * 2 + 1] = acc_l[q][0];
                }
            }
        }
    }
}

constexpr int lds_bytes() { return kRing * kTile + (kPrefillChunkPagesMax + 4) * (int)sizeof(int32_t); }   // ring, page ids of a chunk, the claimed item

}  // namespace prefill

}  // namespace dyn
