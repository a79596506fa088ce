// Shared device helpers for the gfx950 kernels: storage types, bf16 conversion,
// wave-level reductions.  Wavefronts are 64 lanes wide throughout.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace dyn {

typedef uint16_t bf16_t;   // raw bfloat16 storage word

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float(static_cast<uint32_t>(v) << 16); }

// Round to nearest, ties to even.  NaN keeps a quiet payload.
__device__ __forceinline__ bf16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<bf16_t>((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<bf16_t>(u >> 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf2f(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f2bf(v); }

// Butterfly reductions over the 64 lanes of a wave; every lane ends with the result and
// the combination order is fixed by the lane ids.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}

// LDS operand reads as inline assembly, with their waits placed by hand (wait_lgkmcnt).  The compiler's own
// wait insertion waits for every outstanding LDS read before each block of MFMAs, which serialises
// reads and matrix products; reads it does not see it does not wait for.  The price: the compiler
// believes a result is in its registers as soon as the read has been issued, so nothing but
// instructions placed after the matching wait (and a scheduling barrier, where the consumer is not
// assembly itself) may touch them.  LDS operations return in issue order, so "at most N outstanding"
// means everything but the N most recent has arrived; LDS operations the compiler issues in between
// can only make such a wait stricter, never laxer.
template <int OFFSET>
__device__ __forceinline__ bf16x8 lds_read16(unsigned addr) {        // 16 bytes per lane at LDS byte address addr + OFFSET
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds_read offset field");
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
    return v;
}
template <int OFFSET>
__device__ __forceinline__ u32x2 lds_read8(unsigned addr) {          // 8 bytes per lane
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds_read offset field");
    u32x2 v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
    return v;
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {                   // s_waitcnt lgkmcnt(N) only (vmcnt 63, expcnt 7 = no wait)
    static_assert(N >= 0 && N <= 15, "lgkmcnt is a 4-bit counter");
    __builtin_amdgcn_s_waitcnt(0xc07f | (N << 8));
}

// f(integral_constant<int, I0>), ..., f(integral_constant<int, I1 - 1>): a loop whose index is a compile-time
// constant in the body (immediate offsets of the assembly above, register-array indices).
template <int I0, int I1, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I0 < I1) {
        f(std::integral_constant<int, I0>());
        static_for<I0 + 1, I1>(f);
    }
}

// Split-KV chunk size (cached positions per work item) of a query block of a multi-token
// sequence, from `reach` = the largest key count a token of its aligned position block can
// attend.  1024 positions, doubled until the block has at most 8 chunks, up to 8192: behind a
// long cached prefix fixed 1024-position chunks leave one fp32 partial set per 1024 keys and
// token for the merge to read back.  A function of the block's positions alone.
__host__ __device__ inline int prefill_chunk_positions(int reach) {
    int ct = 1024;
    while (reach > 8 * ct && ct < 8192) ct *= 2;
    return ct;
}
constexpr int kPrefillChunkPagesMax = 8192 / 16;     // in 16-position pages
// The same for a block of a long prompt: its sequence has about `rows` tokens in this step with about `mean_keys` keys each, in blocks
// of `tg`, for n_kv kv heads.  Such a prompt has work for all 256 CUs from its query blocks alone, and what a finer cut costs is a
// partial set written and read back per chunk and token: chunks double, to 4096, or to the one chunk of 8192 that holds a whole block,
// while one is at most half of what a CU gets.  Attention,
// chunks of 1024 or 2048 -> these: 4096 tokens alone 247 -> 209 us, behind 2000 positions 433 -> 395, behind 8000 846 -> 801; 6000 behind 2000 651 -> 531.  Beyond, or with
// shorter prompts, what is left over of a CU's last chunk costs more: chunks of 8192 for 4096 tokens behind 8000 positions 812, for 2300 behind 16000
// 712 -> 779, of 4096 for 1200 behind 8000 235 -> 275.  (450 prompts of 10 pairs of head counts, 600 to 10000 tokens behind 0 to 30000 positions: 0.977 of the time
// on average, none longer.)
__host__ __device__ inline int prefill_run_chunk_positions(int reach, int tg, int n_kv, int rows, int mean_keys) {
    int ct = prefill_chunk_positions(reach);
    const long long cu = (long long)n_kv * rows * mean_keys / (256 * tg);
    const int most = reach <= 8192 ? 8192 : 4096;
    while (ct < most && ct < reach && 4 * ct <= cu) ct *= 2;
    return ct;
}
// The chunk size in use: that of the tokens in the aligned block of `tg` positions of a multi-token sequence that row t, at position p, lies in,
// where rows start .. end - 1 are the sequence's (a dispatch holds whole sequences).  A function of that sequence's rows and positions in this
// step, and of nothing else in the dispatch; up to 2560 rows the plain rule.
constexpr int kLongRun = 2560;
__host__ __device__ inline int prompt_chunk_positions(int t, int p, int start, int end, int tg, int n_kv) {
    const int reach = (p / tg + 1) * tg, rows = end - start;
    if (rows <= kLongRun) return prefill_chunk_positions(reach);
    return prefill_run_chunk_positions(reach, tg, n_kv, rows, p - (t - start) + (rows + 1) / 2);
}
// The run of rows, of one sequence, that row `at` of a dispatch of `rows` rows lies in.  count(row, step): how many of the rows row + step, row + 2 step, ..
// row + 64 step are the sequence's, before the first that is not or is no row.  (Up to 64 x 4161 rows to either side: a longer run
// has the longest chunks wherever its ends are.)
struct Run { int start, end; };
template <class Count>
__host__ __device__ inline Run run_around(int at, int rows, Count &&count) {
    int before = 0, after = 0;
    for (int step = rows > 4096 ? 4096 : 64; step >= 1; step /= 64) {
        const int lo = count(at - before, -step), hi = count(at + after, step);
        before += lo * step;
        after += hi * step;
    }
    return Run{at - before, at + after + 1};
}
// The most chunks a token with at most `positions` keys can have under that rule: a chunk size below 8192 is taken up to
// eight chunks' reach only.
__host__ __device__ inline int prefill_max_chunks(long positions) {
    long most = 1;
    for (long ct = 1024; ct <= 8192; ct *= 2) {
        const long keys = ct < 8192 && positions > 8 * ct ? 8 * ct : positions;
        if ((keys + ct - 1) / ct > most) most = (keys + ct - 1) / ct;
    }
    return (int)most;
}

// What a work item does with one of its columns (a token and a q head).  nk: keys the column attends (0: a dead
// column); the item's chunk is the `chunk` positions from `first`, a multiple of `chunk`.  The item of a
// block's later chunk may hold tokens whose keys all lie before it (a block of 16 * (16 / G) positions, 80 at G = 3,
// need not divide the chunk): those are some other item's to write.
enum ColumnEnd { COLUMN_NOT_MINE, COLUMN_DONE, COLUMN_PARTIAL };
__host__ __device__ inline ColumnEnd column_end(int nk, int first, int chunk) {
    if (nk <= first) return COLUMN_NOT_MINE;
    return nk <= chunk ? COLUMN_DONE : COLUMN_PARTIAL;       // one chunk is all: the item writes the output, the merge leaves the token alone
}

// Workgroups, of a launch's `groups`, that start on `items` query blocks while the others start on decodes; prompts, decodes: what the two
// parts cost.  The share that would finish both together if each CU had its part of memory's rate: memory is busy with fewer, so the
// decodes end first, and their workgroups take query blocks after them; the other way round there is no way back.  The share is
// cut to whole rounds of query blocks, which are long beside the launch (2048 tokens beside 64 decodes, 384 of them, on 88 / 112 / 128
// workgroups: 154 / 172 / 148 us).  Up to a quarter of the workgroups each takes one, where the decodes are not long beside it: else as many rounds as a
// fifth of the decodes' time holds, since no workgroup that is through with its query blocks can help with them (attention, apart / one round /
// this: 33 tokens beside 128 decodes of 500 to 4000 positions, 32 kv heads, 32 blocks, 862 / 921 / 867 us; 300 tokens, 64 blocks, 880 / 920 / 876).
// Always down to them: what a workgroup too many takes from the decodes nobody gives back.  To the nearest number of rounds, prompts could
// be left all workgroups but eight, which then had every decode to themselves (attention, launches apart / to the nearest / down, 16 to 40 q heads:
// 300 tokens behind 4000 positions beside 2 decodes of 4000 104 / 406 / 98 us, beside 16 of up to 3000 104 / 353 / 97; 2500 tokens beside 16
// 181 / 415 / 165).  Over 210 mixes (7 pairs of head counts, 33 to 2500 tokens, 2 to 200 decodes), against the best of 18 shares: 1.064 -> 1.028 on
// average.  Against launches apart on the same tensors, over 378 mixes of 9 pairs of head counts: 1.147x on average, the worst 16 and 32 kv heads beside
// 128 decodes of up to 6000 positions, 0.954x (738 -> 773 us).
__host__ __device__ inline int mixed_share(int items, float prompts, float decodes, int groups) {
    const float share = groups * prompts / (prompts + decodes);
    const int whole = share > 1.0f ? (int)share : 1;
    int rounds = (items + whole - 1) / whole;
    if (items <= groups / 4) {
        const float beside = 0.2f * decodes * items / (prompts * groups);
        rounds = beside < rounds ? (beside > 1.0f ? (int)beside : 1) : rounds;
    }
    const int each = ((items + rounds - 1) / rounds + 7) / 8 * 8, most = groups > 8 ? groups - 8 : 0, least = groups / 2 < 8 ? groups / 2 : 8;
    return each < most ? (each > least ? each : least) : most > least ? most : least;
}

}  // namespace dyn
