// Projection kernels whose tile is 256 W rows wide: the many-row launch that folds split-K planes in
// registers.  The tile itself is gemm_tile.h's; here is which workgroup gets which.
#include "gemm_tile.h"

namespace dyn {

// 256 W rows x 128 X rows, planes folded in registers, a ring of three stages (144 KB): the same outputs
// per CU as two 128 x 128 workgroups with a quarter less operand traffic into LDS and two stages
// in flight instead of one, on the hand-laid-out loop.  Bands as in gemm_bf16_kernel.  (Measured: gemm_path.)
__global__ __launch_bounds__(512, 1) void gemm_fold_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                           const bf16_t *__restrict__ R, bf16_t *__restrict__ Y, int M, int N, int K,
                                                           int S, int band) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int n_tile, m_tile;
    if (!band_tile(N / 256, (M + 127) / 128, band, n_tile, m_tile)) return;
    gemm_tile<256, 128, true, 3, false, 8, true>(lds, X, ldx, W, R, Y, N, nullptr, 0, M, N, K, S, nullptr, 1, false, n_tile, 0, m_tile * 128);
}

hipError_t launch_gemm_fold(int grid, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N,
                            int K, int S, int band) {
    constexpr int LDS = 3 * (256 + 128) * ROWB;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_fold_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(gemm_fold_kernel, dim3(grid), dim3(512), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R,
                       (bf16_t *)Y, rows, N, K, S, band);
    return hipGetLastError();
}

}  // namespace dyn
