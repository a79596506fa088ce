// Host-side launch functions of the gfx950 kernels.  Each takes pointers already offset to
// the first token row of the dispatch and the number of rows; none synchronises or
// allocates.  dtype is DYN_F32 (0) or DYN_BF16 (1).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "attn_shape.h"

namespace dyn {

constexpr int kMaxHalfDim = 128;   // rotary tables are passed by value: head_dim <= 256

struct RopeTable {                 // theta_i = base^(-2i/d), i < d/2, computed on the host in fp64
    double inv_freq[kMaxHalfDim];
};

// Expert grouping of a projection (all fields zero: plain GEMM).  Group e has counts[e] rows;
// row i of the group reads X row lists[e * cap + i] / x_div and writes output row
// lists[e * cap + i]; its weights start w_stride elements after the previous group's.
struct GemmGroups {
    const int32_t *counts;
    const int32_t *lists;
    int cap, x_div, n_groups;
    size_t w_stride;
    int force_planes;
};

// Split-K factor of a GEMM with output width N and depth K.  A function of (N, K) alone so
// that a row's summation order never depends on how many rows are in flight.
// Expert-grouped projections multiply `groups` matrices in one launch and need fewer planes each.
int gemm_split_k(int dtype, int N, int K, int groups = 1);
bool gemm_supported(int dtype, int N, int K);
// How launch_gemm runs a plain bf16 projection of `rows` rows (the launcher follows this, and the
// scheduler's cost model prices it).
enum { GEMM_FEW = 0, GEMM_TALL = 1, GEMM_WIDE = 2, GEMM_MANY = 3 };
struct GemmPath {
    int kind;          // GEMM_FEW: 128 x 64|128 tiles, ring of 4; GEMM_TALL: 128 x 256|384|512, eight waves;
                       // GEMM_WIDE: 256 x 256, eight waves; GEMM_MANY: 128 x 128|160, two workgroups per CU, or 256 x 128, one
    int bn, mt;        // tile: W rows x X rows
    int split;         // split-K factor S(N, K)
    bool folded;       // planes accumulated one after another in registers: no plane buffer, no reduce kernel
    int workgroups;    // tiles x planes spread over the grid
    int resident;      // workgroups the chip's 256 CUs hold at a time
    int tail_rows;     // this many last rows run as a launch of their own (its path: gemm_path of that many rows);
                       // workgroups counts the first launch only
};
GemmPath gemm_path(int dtype, int rows, int N, int K);
// True if launch_gemm on `rows` rows writes split-K planes to `partial` (false: one plane, or planes folded in registers).
bool gemm_uses_plane_buffer(int dtype, int rows, int N, int K);

// ld_out: elements between output rows (>= H).
struct GemmRoute;
hipError_t launch_rmsnorm(int dtype, const void *x, const void *g, void *out, int ld_out, int rows, int H, float eps,
                          hipStream_t s, const GemmRoute *route = nullptr);

// What follows a projection on the same token rows and is applied by the same launch sequence,
// so that its input never makes a round trip through a kernel of its own: the RMSNorm of the
// output rows (after the o and down projections) or rotary + cache append (after the qkv
// projection).  Where the projection's split-K planes are summed by a reduce kernel, that kernel
// applies it (one pass over the planes); otherwise the operator's own kernel runs on the rows the
// projection wrote.  Either way every element sees the same arithmetic in the same order.
// The router of the rows that a norm writes (bf16, at most 8 experts), applied behind the norm, by its launch where rows are few: as launch_route, sel and wgt at the first row.  w_router null: none.
struct GemmRoute { const float *w_router = nullptr; int32_t *sel = nullptr; float *wgt = nullptr; int E = 0, top_k = 0; };

struct GemmEpilogue {
    enum { NONE = 0, NORM = 1, ROPE = 2, GATE = 3 } kind = NONE;
    // NORM: h_out[row] = RMSNorm(Y[row]) * g, row pitch ld_h
    // GATE: h_out[row] = silu(first half of Y[row]) * second half, row pitch ld_h; Y is written only where no planes are, and may lie
    // on the plane buffer
    const void *g = nullptr;
    void *h_out = nullptr;
    int ld_h = 0;
    float eps = 0.f;
    GemmRoute route;         // NORM: the router of the normalised rows
    // ROPE: rotary on the q and k heads of the Y rows (q in place), k' and v appended to the cache
    const int32_t *seq_of_token = nullptr, *pos_of_token = nullptr, *block_table = nullptr;
    void *k_cache = nullptr, *v_cache = nullptr;
    const RopeTable *rope = nullptr;
    const AttnShape *shape = nullptr;
    int long_rows = 0;       // of the rows, those of sequences with 16 tokens and more among them
};

// The RMSNorm before a projection, applied to the X rows by the projection itself (g null: none); same bits as launch_rmsnorm's rows.
struct GemmNorm { const void *g = nullptr; float eps = 0.f; };
bool gemm_norm_in_supported(int dtype, int rows, int N, int K, int n_cus);

// Y[rows,N] = X[rows,K] W[N,K]^T (+ R[rows,N]); ldx = elements between rows of X (>= K).  partial: fp32 scratch for split-K planes,
// plane p at partial + p * plane_stride (elements); unused when the split factor is 1.
// If mid is not NULL it is recorded after the contraction kernel, before the split-K reduce.
// n_cus: compute units of the partition the stream runs on, 0: all.
hipError_t launch_gemm(int dtype, const void *X, int ldx, const void *W, const void *R, void *Y, float *partial,
                       size_t plane_stride, int rows, int N, int K, hipStream_t s, hipEvent_t mid = nullptr,
                       const GemmEpilogue *ep = nullptr, int n_cus = 0, const GemmNorm &norm = GemmNorm{});

// fp32 projection, plain or expert-grouped (kernels_gemm_f32.hip; launch_gemm and launch_gemm_grouped call it); max_rows bounds a group's rows.
hipError_t launch_gemm_f32(const void *X, int ldx, const void *W, const void *R, void *Y, int max_rows, int N, int K, const GemmGroups &gr,
                           hipStream_t s);
bool gemm_f32_gated_supported(int N2, int K);
bool gemm_f32_rope_supported(const void *X, int ldx, const void *W, int rows, int N, int K, const AttnShape &sh);   // rotary + cache append in the same launch
hipError_t launch_gemm_f32_rope(const void *X, int ldx, const void *W, void *Y, int rows, int N, int K, const GemmNorm &norm, const GemmEpilogue &rope,
                                hipStream_t s);
bool gemm_f32_gated_rows_supported(int rows, int N2, int K);         // with that many rows, or any
bool gemm_f32_norm_supported(int rows, int N, int K, int n_cus);     // with rotary or gate, the norm of X in the same launch
hipError_t launch_gemm_f32_gated(const void *X, int ldx, const void *W, void *Y, int ldy, int rows, int N2, int K, const GemmNorm &norm, hipStream_t s);
// A few rows (at most 16), planes summed in the workgroup (kernels_gemm_rows.hip; launch_gemm calls it).
bool gemm_rows16_wide_supported(int rows, int N, int K, int S);       // on the whole chip
bool gemm_rows16_supported(int rows, int N, int K, int S);            // on any number of CUs
bool gemm_rows16_taken(int rows, int N, int K, int S, int n_cus, bool norm);   // n_cus: of the partition, 0: all; norm: an RMSNorm follows
bool gemm_rows16_rope_supported(const AttnShape &sh);                 // with rotary + cache append in the same launch
hipError_t launch_gemm_rows16(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S,
                              const GemmEpilogue *rope);
// Many rows, split-K planes folded in registers, 256 x 128 tiles (kernels_gemm_wide.hip; launch_gemm calls it).
hipError_t launch_gemm_fold(int grid, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N,
                            int K, int S);
// The same rows without planes, on 256-wide tiles of several heights: tiles[i] m tiles of 64 (i + 1) rows.  wide_cut: the heights for a launch, if they
// beat `now` (in rounds of 256 x 256 tiles); rows x N has to be GEMM_WIDE's.
struct WideCut { int tiles[4]; };
bool wide_cut(int rows, int N, float now, WideCut *out);
bool gemm_cut(const GemmPath &p, int rows, int N, int n_cus, WideCut *cut);   // whether launch_gemm and launch_gemm_gated take them for p, on n_cus CUs (0: all)
float cut_rounds(const WideCut &cut, int N);                                  // the longest CU's share, in rounds of 256 x 256 tiles
hipError_t launch_gemm_cut(bool gated, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int ldy, int rows, int N, int K,
                           const WideCut &cut);
// Gate/up with planes folded in registers and the gate in the epilogue (bf16): the tile height for a launch, 0 where planes go over workgroups.
int gate_fold_rows(int rows, int N2, int K);
bool gate_fold_taken(int rows, int N2, int K, int n_cus);              // on n_cus CUs, 0: all
hipError_t launch_gemm_gate_fold(hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, int rows, int N2, int K);
// Planes folded in registers, 128-wide tiles of several heights: tiles[i] m tiles of 96 + 32 i rows.  fold_cut: the heights for a launch, if they beat
// p's one.
struct FoldCut { int tiles[3]; };
bool fold_cut(const GemmPath &p, int rows, int N, FoldCut *out);     // with weights that stay in the last-level cache
bool gemm_fold_cut(const GemmPath &p, int rows, int N, int K, int n_cus, FoldCut *out);
float cut_rounds(const FoldCut &cut, int N);                         // the longest CU's share, in rounds of two 128 x 128 tiles a CU
hipError_t launch_gemm_fold_cut(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S,
                                const FoldCut &cut);
// Expert-grouped projection without planes on 256-wide tiles of a height chosen per expert (the grouped launchers
// call it); gated: silu(gate) * up to Y, else Y, or fp32 to P with gr.force_planes.
hipError_t launch_gemm_experts_wide(bool gated, hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, float *P, int N,
                                    int K, const GemmGroups &gr);
// The same on 128-wide tiles, with or without planes (plane p of S at P + p * plane_stride where there are several or gr.force_planes).
hipError_t launch_gemm_experts(bool gated, hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, float *P, size_t plane_stride,
                               int max_rows, int N, int K, int S, const GemmGroups &gr);

hipError_t launch_gemm_grouped(int dtype, const void *X, int ldx, const void *W, void *Y, float *partial,
                               size_t plane_stride, const GemmGroups &gr, int max_rows, int row0, int n_rows, int N, int K,
                               hipStream_t s, hipEvent_t mid = nullptr);

// Gate/up projection with the SiLU gate applied in the epilogue (bf16: split factor 1 only; fp32: not expert-grouped):
// Y[row, N2/2] = silu(X Wg^T) * (X Wu^T), row pitch ldy.  gr.n_groups = 0: plain, pointers offset to
// the dispatch's first row, max_rows rows.  Grouped: as launch_gemm_grouped.
bool gemm_gated_supported(int dtype, int N2, int K, bool experts);
hipError_t launch_gemm_gated(int dtype, const void *X, int ldx, const void *W, void *Y, int ldy, const GemmGroups &gr, int max_rows,
                             int N2, int K, hipStream_t s, hipEvent_t mid = nullptr, const GemmNorm &norm = GemmNorm{}, int n_cus = 0);

// MoE router for token rows: logits = h W_r^T in fp32, top_k largest (ties to the lower index),
// softmax over the selected logits.  sel / wgt are [rows, top_k], largest logit first.
hipError_t launch_route(int dtype, const void *h, int ldh, const float *w_router, int32_t *sel, float *wgt, int rows,
                        int H, int E, int top_k, hipStream_t s);

// Per-expert lists of (token, rank) pairs p = t * top_k + j in ascending p, for the rows of one
// dispatch: counts[E], lists[E, cap].  pair_base = first pair id of the dispatch.
bool expert_lists_scan(int n_pairs, int E);      // by a wave per expert, else by sixteen waves
hipError_t launch_expert_lists(const int32_t *sel, int n_pairs, int pair_base, int E, int cap, int32_t *counts,
                               int32_t *lists, hipStream_t s);

// y[t] = x2[t] + sum_j wgt[t, j] * (sum_p planes[p][t * top_k + j]) in rank order j, planes in order p.
hipError_t launch_moe_combine(int dtype, const float *planes, size_t plane_stride, int S, const float *wgt,
                              const void *x2, void *y, int rows, int H, int top_k, hipStream_t s);

// Rotary on the q and k heads of qkv rows (in place for q) and cache append of k', v.
hipError_t launch_rope_kv(int dtype, void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                          const int32_t *block_table, void *k_cache, void *v_cache, const RopeTable &tab,
                          const AttnShape &sh, int rows, int long_rows, hipStream_t s);

// The attention work lists inside `plan` (scratch of (4 * max_chunks + 5) * rows + 4 int32 at most): single-token
// sequences, multi-token sequences, and the chunk size every token's partials are indexed by.
struct AttnPlan { int32_t *single, *multi, *ct_of_token; };
AttnPlan attn_plan_lists(int32_t *plan, const AttnShape &sh, int rows);
bool attention_mfma_supported(int dtype, const AttnShape &sh);      // the shapes whose attention walks these lists
int attn_prefill_max_chunks(long positions);      // the most chunks its prompt form cuts a token's keys into
hipError_t launch_attn_plan(const int32_t *seq_of_token, const int32_t *pos_of_token, int32_t *plan, const AttnShape &sh, int rows, hipStream_t s);
// The lists of some rows and the RMSNorm of the same rows (bf16) in one launch: neither needs the other.
hipError_t launch_norm_plan(const void *x, const void *g, void *out, int ld_out, int rows, int H, float eps, const int32_t *seq_of_token,
                            const int32_t *pos_of_token, int32_t *plan, const AttnShape &sh, hipStream_t s);

// Causal paged attention for token rows; part_o / part_ml are the split-KV partial arrays
// ([rows, max_chunks, n_q, head_dim] and [rows, max_chunks, n_q, 2], part_index); plan is scratch for the
// device-built work lists (AttnPlan); any_single / any_multi: some sequence has one / more
// than one token in these rows (host knowledge; whether the decode / the prefill form is launched).
hipError_t launch_attention(int dtype, const void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                            const int32_t *block_table, const void *k_cache, const void *v_cache, void *out, int ld_out,
                            float *part_o, float *part_ml, int32_t *plan, bool any_single, bool any_multi, const AttnShape &sh,
                            int rows, hipStream_t s, hipEvent_t mid = nullptr,    // mid: recorded between the chunk kernel and the combine
                            hipEvent_t pre = nullptr,   // pre: recorded after the work-list kernel, before the chunk kernel
                            bool plan_ready = false);   // `plan` already holds the lists of these rows (built by the first norm's launch or an earlier layer's call)

// The same from a gate/up projection's split-K planes ([rows, 2 I] each): summed in plane order, rounded to bf16, gated.
bool reduce_gate_supported(int dtype, int I);
hipError_t launch_reduce_gate(const float *P, size_t plane_stride, int S, void *out, int ld_out, int rows, int I, hipStream_t s);
// out[rows, I] = silu(gu[:, :I]) * gu[:, I:]
hipError_t launch_silu_mul(int dtype, const void *gu, void *out, int ld_out, int rows, int I, hipStream_t s);

// The split-K reduce of a projection fused with what follows it (bf16; used by launch_gemm).
hipError_t launch_reduce_norm(const float *P, size_t plane_stride, int S, const void *R, void *Y, const void *g, void *out,
                              int ld_out, int rows, int H, float eps, hipStream_t s, const GemmRoute *route = nullptr);
bool reduce_rope_supported(int dtype, const AttnShape &sh);
hipError_t launch_reduce_rope(const float *P, size_t plane_stride, int S, void *qkv, const int32_t *seq_of_token,
                              const int32_t *pos_of_token, const int32_t *block_table, void *k_cache, void *v_cache,
                              const RopeTable &tab, const AttnShape &sh, int rows, hipStream_t s);

// Measurement aid: reads `bytes` (a multiple of 16, 16-byte aligned) of buf once; sink receives 8192 words.
hipError_t launch_stream_read(const void *buf, size_t bytes, uint32_t *sink, hipStream_t s);
// Matrix-core probe (kernels_gemm.hip): n_stages stages of the wide projection tile's main loop on 256 workgroups,
// operands from the first mfma_probe_bytes() of buf; sink takes 256 x 512 floats.
size_t mfma_probe_bytes();
double mfma_probe_flops(int n_stages);
hipError_t launch_mfma_probe(const void *buf, int n_stages, float *sink, hipStream_t s);

}  // namespace dyn
