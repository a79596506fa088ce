// The attention's shape and where its partial results lie.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace dyn {

struct AttnShape {
    int n_q, n_kv, head_dim, page_size;
    int max_pages_per_seq;         // block-table row length
    int chunk_pages;               // pages per split-KV chunk (a constant of the layer)
    int max_chunks;                // the most chunks a token of the batch can have
    int n_cus;                     // CUs of the stream's partition (0: whole device); sizes the persistent launch
};

// Where chunk c of a row's q head lies in the split-KV partial arrays: a token's chunks behind one another, the heads of one side by side, so
// what is written at one time - a few tokens' chunks - is one piece of memory.  (Chunk by chunk over all rows, a token's chunks lay a
// whole number of MiB apart: 256 tokens of up to 32 chunks, attention 861 us where this takes 858, three layers' step 3198 -> 3176.)
__host__ __device__ inline size_t part_index(const AttnShape &sh, int row, int head, int c) { return ((size_t)row * sh.max_chunks + c) * sh.n_q + head; }

}  // namespace dyn
