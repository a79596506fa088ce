// The work lists of paged attention (bf16, head_dim 128, 16-position pages), built on the device, and the
// launch that builds them beside the first norm.
#include "common.h"
#include "kernels.h"
#include "norm_row.h"

namespace dyn {

int attn_prefill_block_tokens(const AttnShape &sh);

constexpr int PS = 16;

// Work lists, built on the device from the positions (contexts differ by 8x inside a batch, so
// a dense token x max_chunks grid would be mostly empty workgroups).  A wave serves a query
// group: tokens of one sequence whose positions fall in the same aligned block of `tg`
// positions, all of them against one pass over the keys.  List 0 holds the tokens that are
// alone in their sequence this step (decode: groups of one, 4 of 16 MFMA columns live), list 1
// the tokens of multi-token sequences (prefill chunks) in query blocks of up to tg1 tokens, against
// chunks of prompt_chunk_positions() positions (1024 unless the block reaches past 8192 keys; more for a long prompt).
// One entry per (group, chunk) that exists: list[0] = number of entries, entry i =
// (first token row, chunk | tokens << 20) at list[2 + 2 i].
// List 0 is ordered by work, largest first: its entries are bucketed by their size in quarters of
// the largest chunk (kPlanBuckets buckets; with the default chunk of 16 pages a quarter is one
// tile pair of four pages) and inside a bucket they stay in token order, so the eight kv heads of a chunk and the chunks
// of a sequence remain neighbours.  The persistent decode kernel deals the list out by wave index
// in a snake (attn_mfma_kernel): with equal-sized items first and the small ones at the end, the
// waves' totals differ by about one percent instead of six on contexts spread over 1024..8192.
//
// One workgroup of 16 waves walks the rows 1024 at a time.  A sequence's tokens are adjacent rows with
// consecutive positions, so a token leads its group iff it starts its sequence or its aligned block.
// Entry offsets come from a wave scan plus one LDS step per list (per bucket of list 0).  What it costs is the
// latency of its dependent loads, so a batch's rows are classified once (kBatches batches are kept
// in registers for the second pass), a group's size is first tried as the whole block, and the launch
// does not stand alone: the layer's first norm, which nothing of this depends on, runs in the same grid
// (norm_plan_kernel).  Lists + norm as two launches -> this one: 1 token 10.2 -> 5.7 us, 128 tokens 11.0 -> 7.3,
// 2112 rows 27.6 -> 17.8, 4096 rows 43.6 -> 25.3 us.
constexpr int kPlanBuckets = 4, kBatches = 4;

// Inclusive sums over the 64 lanes and over each row of 16 lanes, on the vector ALU (a shuffle goes through LDS: five
// scans of six shuffles were a third of the lists' time).
__device__ __forceinline__ int scan16(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    return x;
}
__device__ __forceinline__ int scan64(int x) {
    x = scan16(x);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast 15: rows 1 and 3 take the row below's total
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // row_bcast 31: rows 2 and 3 take lane 31's
    return x;
}

struct PlanRow { int which, nc, n_tok, b_full, b_last; };

// LONG: a dispatch that may hold a prompt of more than kLongRun rows.  Without the search for one, and the rows past kBatches, the launch is half as
// long in code (norm and lists 34 -> 18 KB), which a kernel that runs once a step has to fetch first: one token's step 118.0 -> 116.5 us, 128 decodes
// 401.3 -> 400.7.
template <bool LONG>
__device__ __forceinline__ void attn_plan(const int32_t *__restrict__ seq_of_token, const int32_t *__restrict__ pos_of_token, int rows, int ct,
                                          int tg1, int n_kv, int32_t *__restrict__ plan0, int32_t *__restrict__ plan1,
                                          int32_t *__restrict__ ct_of_token) {
    constexpr int NL = kPlanBuckets + 1;                    // scanned counters: list 0's buckets, then list 1
    __shared__ int wave_tot[NL][16];
    __shared__ int bucket_total[kPlanBuckets];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk_pages = ct / PS, bucket_pages = max(1, (chunk_pages + kPlanBuckets - 1) / kPlanBuckets);

    // The rows of the sequence that row t belongs to, as far as they matter: a sequence of more than kLongRun rows has the first or the last of a
    // wave's 64 rows, so the wave looks for the ends of those two, 64 rows at a time, unless its last rows were of the same.  All lanes call this.
    // (A lane for itself, in steps around its block: lists and norm of 4096 / 8192 rows 24 / 39 -> 29 / 53 us in 8 steps, 31 / 70 in 20; this 27 / 44.)
    Run known{0, 0};
    auto run_of = [&](int t) {
        Run run{t, t + 1};
        if constexpr (LONG) {
            const int first = __builtin_amdgcn_readfirstlane(t);
            if (first >= rows) return run;
            for (int edge : {first, min(first + 63, rows - 1)}) {
                if (edge < known.start || edge >= known.end) {
                    const int s = seq_of_token[edge];
                    known = run_around(edge, rows, [&](int row, int step) {
                        const int r = row + step * (lane + 1);
                        return (int)__popcll(__ballot(r >= 0 && r < rows && seq_of_token[min(max(r, 0), rows - 1)] == s));
                    });
                }
                if (t >= known.start && t < known.end) run = known;
            }
        }
        return run;
    };

    // What token row t contributes: which list, how many entries, and for list 0 the buckets of
    // its chunks (all but the last have the sequence's balanced chunk size, the last the rest).
    auto classify = [&](int t, const Run &run) {
        PlanRow r{0, 0, 0, 0, 0};
        const int before = max(t - 1, 0), after = min(t + 1, rows - 1);
        const int s = seq_of_token[t], s_before = seq_of_token[before], s_after = seq_of_token[after], p = pos_of_token[t];
        const bool prev_same = t > 0 && s_before == s, next_same = t + 1 < rows && s_after == s;
        r.which = prev_same || next_same;
        const int tg = r.which ? tg1 : 1, ctw = r.which ? prompt_chunk_positions(t, p, run.start, run.end, tg1, n_kv) : ct;
        if (!prev_same || p % tg == 0) {                     // group leader
            const int cand = min(tg - p % tg, rows - t);     // positions left in the aligned block
            // rows t .. t + n_tok - 1 belong to the sequence: the matches form a prefix of the
            // candidates, mostly all of them, else found by bisection
            int lo = 1, hi = cand;                           // n_tok lies in [lo, hi]
            if (cand > 1 && seq_of_token[t + cand - 1] == s) lo = hi;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (seq_of_token[t + mid - 1] == s) lo = mid;
                else hi = mid - 1;
            }
            r.n_tok = lo;
            r.nc = (p + r.n_tok - 1 + ctw) / ctw;            // chunks the group's last token reaches
            if (!r.which) {                                  // the decode kernel's own chunking of this sequence
                const int seq_pages = (p + PS) / PS;         // ceil((p + 1) / PS)
                const int cp = (seq_pages + r.nc - 1) / r.nc, last = seq_pages - (r.nc - 1) * cp;
                r.b_full = max(0, kPlanBuckets - (cp + bucket_pages - 1) / bucket_pages);
                r.b_last = max(0, kPlanBuckets - (last + bucket_pages - 1) / bucket_pages);
            }
        }
        ct_of_token[t] = ctw;                                // the chunk size this token's partials are indexed by
        return r;
    };

    // pass 1: sizes of list 0's buckets
    if (threadIdx.x < kPlanBuckets) bucket_total[threadIdx.x] = 0;
    __syncthreads();
    PlanRow kept[kBatches];
    auto count = [&](const PlanRow &r) {
        if (!r.which && r.nc > 0) {
            if (r.nc > 1) atomicAdd(&bucket_total[r.b_full], r.nc - 1);
            atomicAdd(&bucket_total[r.b_last], 1);
        }
    };
#pragma unroll
    for (int b = 0; b < kBatches; ++b) {
        const int t = b * 1024 + (int)threadIdx.x;
        kept[b] = PlanRow{0, 0, 0, 0, 0};
        const Run run = run_of(t);
        if (t < rows) kept[b] = classify(t, run);
    }
#pragma unroll
    for (int b = 0; b < kBatches; ++b) count(kept[b]);
    for (int t0 = kBatches * 1024; LONG && t0 < rows; t0 += 1024) {
        const int t = t0 + (int)threadIdx.x;
        const Run run = run_of(t);
        if (t < rows) count(classify(t, run));
    }
    __syncthreads();
    int base[NL];                                             // next free entry of each bucket / of list 1
    base[0] = 0;
#pragma unroll
    for (int k = 1; k < kPlanBuckets; ++k) base[k] = base[k - 1] + bucket_total[k - 1];
    const int total0 = base[kPlanBuckets - 1] + bucket_total[kPlanBuckets - 1];
    base[kPlanBuckets] = 0;

    // pass 2: entries, in token order inside each bucket
    auto place = [&](int t, const PlanRow &r) {
        int v[NL];                                            // this thread's entries per counter
#pragma unroll
        for (int k = 0; k < NL; ++k) v[k] = 0;
        if (r.which) {
            v[kPlanBuckets] = r.nc;
        } else if (r.nc > 0) {
#pragma unroll
            for (int k = 0; k < kPlanBuckets; ++k) v[k] = (k == r.b_full ? r.nc - 1 : 0) + (k == r.b_last ? 1 : 0);
        }
        int incl[NL];                                         // inclusive wave scans
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int x = scan64(v[k]);
            incl[k] = x;
            if (lane == 63) wave_tot[k][wave] = x;
        }
        __syncthreads();
        int start[NL];
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int sums = scan16(wave_tot[k][lane & 15]);
            const int pre = wave ? __builtin_amdgcn_readlane(sums, wave - 1) : 0, tot = __builtin_amdgcn_readlane(sums, 15);
            start[k] = base[k] + pre + incl[k] - v[k];
            base[k] += tot;
        }
        if (r.which) {
            for (int c = 0; c < r.nc; ++c) {
                plan1[2 + 2 * (start[kPlanBuckets] + c)] = t;
                plan1[3 + 2 * (start[kPlanBuckets] + c)] = c | (r.n_tok << 20);
            }
        } else if (r.nc > 0) {
            int at_full = 0, at_last = 0;
#pragma unroll
            for (int k = 0; k < kPlanBuckets; ++k) {          // select without indexing the register arrays dynamically
                if (k == r.b_full) at_full = start[k];
                if (k == r.b_last) at_last = start[k] + (r.b_last == r.b_full ? r.nc - 1 : 0);
            }
            for (int c = 0; c + 1 < r.nc; ++c) {
                plan0[2 + 2 * (at_full + c)] = t;
                plan0[3 + 2 * (at_full + c)] = c | (1 << 20);
            }
            plan0[2 + 2 * at_last] = t;
            plan0[3 + 2 * at_last] = (r.nc - 1) | (1 << 20);
        }
        __syncthreads();                                      // wave_tot is reused by the next batch
    };
#pragma unroll
    for (int b = 0; b < kBatches; ++b)
        if (b * 1024 < rows) place(b * 1024 + (int)threadIdx.x, kept[b]);
    for (int t0 = kBatches * 1024; LONG && t0 < rows; t0 += 1024) {
        const int t = t0 + (int)threadIdx.x;
        const Run run = run_of(t);
        place(t, t < rows ? classify(t, run) : PlanRow{0, 0, 0, 0, 0});
    }
    if (threadIdx.x == 0) { plan0[0] = total0; plan1[0] = base[kPlanBuckets]; plan1[1] = 0; }   // list sizes; list 1's work counter
}

static_assert(kLongRun <= kBatches * 1024, "the short form keeps all its rows");

template <bool LONG>
__global__ __launch_bounds__(1024) void attn_plan_kernel(const int32_t *__restrict__ seq_of_token, const int32_t *__restrict__ pos_of_token, int rows,
                                                         int ct, int tg1, int n_kv, int32_t *__restrict__ plan0, int32_t *__restrict__ plan1,
                                                         int32_t *__restrict__ ct_of_token) {
    attn_plan<LONG>(seq_of_token, pos_of_token, rows, ct, tg1, n_kv, plan0, plan1, ct_of_token);
}

// Workgroup 0 builds the lists, each of the others normalises four rows.
template <bool LONG>
__global__ __launch_bounds__(1024) void norm_plan_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ g, bf16_t *__restrict__ out, int ld_out,
                                                         int H, float eps, const int32_t *__restrict__ seq_of_token,
                                                         const int32_t *__restrict__ pos_of_token, int rows, int ct, int tg1, int n_kv,
                                                         int32_t *__restrict__ plan0, int32_t *__restrict__ plan1,
                                                         int32_t *__restrict__ ct_of_token) {
    if (blockIdx.x == 0) {
        attn_plan<LONG>(seq_of_token, pos_of_token, rows, ct, tg1, n_kv, plan0, plan1, ct_of_token);
        return;
    }
    __shared__ float part[4][4];
    const int mine = threadIdx.x >> 8, row = (int)(blockIdx.x - 1) * 4 + mine;
    rmsnorm_row<bf16_t>(x + (size_t)row * H, g, out + (size_t)row * ld_out, H, eps, threadIdx.x & 255, part[mine], row < rows);
}

AttnPlan attn_plan_lists(int32_t *plan, const AttnShape &sh, int rows) {
    const size_t entries = (size_t)rows * sh.max_chunks;
    return AttnPlan{plan, plan + 2 + 2 * entries, plan + 4 + 4 * entries};
}

hipError_t launch_attn_plan(const int32_t *seq_of_token, const int32_t *pos_of_token, int32_t *plan, const AttnShape &sh, int rows, hipStream_t s) {
    const AttnPlan l = attn_plan_lists(plan, sh, rows);
    hipLaunchKernelGGL(rows > kLongRun ? attn_plan_kernel<true> : attn_plan_kernel<false>, dim3(1), dim3(1024), 0, s, seq_of_token, pos_of_token, rows, sh.chunk_pages * PS,
                       attn_prefill_block_tokens(sh), sh.n_kv, l.single, l.multi, l.ct_of_token);
    return hipGetLastError();
}

hipError_t launch_norm_plan(const void *x, const void *g, void *out, int ld_out, int rows, int H, float eps, const int32_t *seq_of_token,
                            const int32_t *pos_of_token, int32_t *plan, const AttnShape &sh, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const AttnPlan l = attn_plan_lists(plan, sh, rows);
    hipLaunchKernelGGL(rows > kLongRun ? norm_plan_kernel<true> : norm_plan_kernel<false>, dim3(1 + (rows + 3) / 4), dim3(1024), 0, s, (const bf16_t *)x, (const bf16_t *)g, (bf16_t *)out, ld_out, H, eps,
                       seq_of_token, pos_of_token, rows, sh.chunk_pages * PS, attn_prefill_block_tokens(sh), sh.n_kv, l.single, l.multi, l.ct_of_token);
    return hipGetLastError();
}

}  // namespace dyn
