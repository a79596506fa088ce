// Projection kernels whose tile is 256 W rows wide or chosen per expert on the device: the many-row
// launch that folds split-K planes in registers, and the expert-grouped launches.  The tile itself is
// gemm_tile.h's; here is which workgroup gets which.
#include <algorithm>

#include "gemm_tile.h"

namespace dyn {

// 256 W rows x 128 X rows, planes folded in registers, a ring of three stages (144 KB): the same outputs
// per CU as two 128 x 128 workgroups with a quarter less operand traffic into LDS and two stages
// in flight instead of one, on the hand-laid-out loop.  Bands as in gemm_bf16_kernel.  (Where they pay, measured: fold_tiles.)
__global__ __launch_bounds__(512, 1) void gemm_fold_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                           const bf16_t *__restrict__ R, bf16_t *__restrict__ Y, int M, int N, int K,
                                                           int S) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int n_tile, m_tile;
    if (!band_tile(N / 256, (M + 127) / 128, gemm_band(M, N, K), n_tile, m_tile)) return;
    gemm_tile<256, 128, true, 3, false, 8, true>(lds, X, ldx, W, R, Y, N, nullptr, 0, M, N, K, S, nullptr, 1, false, n_tile, 0, m_tile * 128, 0);
}

hipError_t launch_gemm_fold(int grid, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N,
                            int K, int S) {
    constexpr int LDS = 3 * (256 + 128) * ROWB;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_fold_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(gemm_fold_kernel, dim3(grid), dim3(512), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R,
                       (bf16_t *)Y, rows, N, K, S);
    return hipGetLastError();
}

// Expert-grouped launch with 256 W rows per tile, for some hundred rows per expert (no planes).  The host
// knows the number of (token, expert) pairs but not how they fall on the experts; a tile height fixed
// on the host computes up to 255 rows of padding per expert.  Here every expert's rows are cut into as few m tiles as hold them, of
// whole 64s, and the workgroup runs one of four bodies.  A launch of several rounds is as long as its work: up to 256 rows a tile
// and heights that add up to the rows (5 x 64 rows: 192 + 128).  One round is as long as its tallest tile: the
// lowest bodies that still run at once, an expert's tiles alike (they stay in step on W).  The experts with the tallest
// tiles come first and the short ones fill the end of the launch; an expert's tiles stay together whatever
// their heights (apart, W came from memory twice: gate/up 601 -> 625 us).  XCD u takes the n tiles congruent to u for all
// experts, an m tile's n tiles in a row (they share X).
// Measured against 256 x 256 tiles throughout (8 experts of a skewed router, two per token): 1100 / 1500 / 2048
// tokens, gate/up 668 / 1006 / 1203 -> 611 / 852 / 1077 us, down 412 / 700 / 765 -> 410 / 421 / 720 us.  Against equal tiles of up to 256
// rows in every launch, 1120 tokens of four seeds: gate/up 611, 703, 701, 620 -> 608, 671, 665, 601 us, down 415, 411, 405, 416 -> 380, 417, 411, 413
// (the first alone fits lower tiles in its round).
constexpr int kExpertsBN = 256, kXcdCus = 32;
constexpr int kExpertsLds = 160 * 1024;               // the bodies' rings: 2 x 64, 2 x 56, 3 x 48, 4 x 40 KB

template <bool GATED>
__global__ __launch_bounds__(512, 1) void gemm_experts_wide_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                                   bf16_t *__restrict__ Y, int ldy, float *__restrict__ P, int N, int K,
                                                                   GemmGroups gr) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int u = blockIdx.x % 8, v = blockIdx.x / 8, nt = N / kExpertsBN;
    const int n_local = (nt - u + 7) / 8;             // n tiles u, u + 8, ...
    if (n_local <= 0) return;
    // Every wave holds the counts, one a lane.  The tallest body a tile may take: the lowest with which this XCD's tiles all run at
    // once, 256 rows if none.
    const int counts = (int)(threadIdx.x & 63) < gr.n_groups ? gr.counts[threadIdx.x & 63] : 0;
    int n2 = 0, n3 = 0, n4 = 0, n1 = 0;
    for (int e = 0; e < gr.n_groups; ++e) {
        const int all = (__builtin_amdgcn_readlane(counts, e) + 63) / 64;
        n1 += all; n2 += (all + 1) / 2; n3 += (all + 2) / 3; n4 += (all + 3) / 4;
    }
    const int fit = kXcdCus / n_local;
    const int top = n1 <= fit ? 1 : n2 <= fit ? 2 : n3 <= fit ? 3 : 4;
    const bool once = n4 <= fit;                       // one round: as long as its tallest tile, which equal tiles keep low and in step on W
    int m = v / n_local, e = 0, units = 0, rows = 0, m0 = 0;   // m: place of the m tile in launch order
    const int n_tile = (v - m * n_local) * 8 + u;
    bool found = false;
    for (int size = top; size >= 1 && !found; --size)   // m tiles of 64 * size rows
        for (e = 0; e < gr.n_groups; ++e) {
            rows = __builtin_amdgcn_readlane(counts, e);
            const int all = (rows + 63) / 64, n_m = (all + top - 1) / top;
            if (n_m == 0) continue;
            const int low = once ? ((rows + n_m - 1) / n_m + 63) / 64 : all / n_m, taller = once ? 0 : all - low * n_m;   // the first `taller` m tiles are 64 rows taller
            if (size != low + (taller > 0)) continue;
            if (m < n_m) {
                units = low + (m < taller);
                m0 = 64 * (m * low + min(m, taller));
                found = true;
                break;
            }
            m -= n_m;
        }
    if (!found || m0 >= rows) return;                  // equal tiles of whole 64s may leave the last one empty
    const int32_t *list = gr.lists + (size_t)e * gr.cap;
    const bf16_t *We = W + (size_t)e * gr.w_stride;
#define DYN_BODY(MT, NS) gemm_tile<kExpertsBN, MT, false, NS, GATED, 8, true>(lds, X, ldx, We, nullptr, Y, ldy, P, 0, rows, N, K, 1, list, gr.x_div, gr.force_planes, n_tile, 0, m0, e)
    if (units == 4) DYN_BODY(256, 2);
    else if (units == 3) DYN_BODY(192, 2);
    else if (units == 2) DYN_BODY(128, 3);
    else DYN_BODY(64, 4);
#undef DYN_BODY
}

hipError_t launch_gemm_experts_wide(bool gated, hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, float *P, int N,
                                    int K, const GemmGroups &gr) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_experts_wide_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kExpertsLds);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_experts_wide_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kExpertsLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    // per XCD: at most one partly filled 256-row m tile per expert, or lower tiles that fit its CUs; workgroups past the last tile end at once
    const int m_tiles = gr.cap / 256 + gr.n_groups, grid = 8 * std::max((N / kExpertsBN + 7) / 8 * m_tiles, kXcdCus);
    if (gated)
        hipLaunchKernelGGL(gemm_experts_wide_kernel<true>, dim3(grid), dim3(512), kExpertsLds, s, (const bf16_t *)X, ldx, (const bf16_t *)W,
                           (bf16_t *)Y, ldy, P, N, K, gr);
    else
        hipLaunchKernelGGL(gemm_experts_wide_kernel<false>, dim3(grid), dim3(512), kExpertsLds, s, (const bf16_t *)X, ldx, (const bf16_t *)W,
                           (bf16_t *)Y, ldy, P, N, K, gr);
    return hipGetLastError();
}

}  // namespace dyn
