// The launch for the tokens of multi-token sequences alone (attn_prefill.h; beside decodes: attn_mixed_kernel).
#include "attn_prefill.h"

namespace dyn {

__global__ __launch_bounds__(prefill::kWaves * 64, 1) void attn_prefill_kernel(const bf16_t *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                                     const int32_t *__restrict__ pos_of_token, const int32_t *__restrict__ block_table,
                                                                     const bf16_t *__restrict__ k_cache, const bf16_t *__restrict__ v_cache,
                                                                     bf16_t *__restrict__ out, int ld_out, float *__restrict__ part_o,
                                                                     float *__restrict__ part_ml, AttnShape sh, const int32_t *__restrict__ plan,
                                                                     int32_t *__restrict__ counter, const int32_t *__restrict__ ct_of_token) {
    prefill::attn_prefill_items(qkv, seq_of_token, pos_of_token, block_table, k_cache, v_cache, out, ld_out, part_o, part_ml, sh, plan, counter, ct_of_token);
}

int attn_prefill_max_chunks(long positions) { return prefill_max_chunks(positions); }

int attn_prefill_block_tokens(const AttnShape &sh) { return prefill::kWaves * prefill::kSets * (16 / (sh.n_q / sh.n_kv)); }

hipError_t launch_attention_prefill(const void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                                    const int32_t *block_table, const void *k_cache, const void *v_cache, void *out, int ld_out,
                                    float *part_o, float *part_ml, const AttnShape &sh, int32_t *plan, const int32_t *ct_of_token, long max_items, int max_groups,
                                    hipStream_t s) {
    static_assert(kPrefillChunkPagesMax <= prefill::kWaves * 64, "one thread per page id of a chunk");
    constexpr int lds_bytes = prefill::lds_bytes();
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)attn_prefill_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int grid = (int)(max_items < max_groups ? max_items : max_groups);
    hipLaunchKernelGGL(attn_prefill_kernel, dim3(grid), dim3(prefill::kWaves * 64), lds_bytes, s, (const bf16_t *)qkv, seq_of_token,
                       pos_of_token, block_table, (const bf16_t *)k_cache, (const bf16_t *)v_cache, (bf16_t *)out, ld_out, part_o, part_ml, sh, plan,
                       plan + 1, ct_of_token);
    return hipGetLastError();
}

}  // namespace dyn
