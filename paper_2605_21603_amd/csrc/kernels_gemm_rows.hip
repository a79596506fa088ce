// bf16 projections with planes for a few rows: the planes summed inside the workgroup.
#include <hip/hip_runtime.h>

#include "gemm_tile.h"
#include "kernels.h"

namespace dyn {

// A workgroup owns 16 W rows over the whole depth, wave p plane p of the S; a lane loads its MFMA operands straight into
// registers, kDeep stages ahead, and the planes meet in LDS.  Bound by the weight stream; what it saves is the planes'
// way through memory and the launch that sums them.  The stages of a plane are walked in the rotated order of
// the other tiles and the planes are added in plane order: the same bits.
constexpr int kDeep = 8;

template <int S>
__global__ __launch_bounds__(64 * S) void gemm_rows16_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                             const bf16_t *__restrict__ R, bf16_t *__restrict__ Y, int rows,
                                                             int N, int K) {
    __shared__ f32x4 planes[S][64];
    const int lane = threadIdx.x & 63, sp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
    const int n0 = blockIdx.x * 16, Kp = K / S, n_stage = Kp / 64;
    const int rot = (int)(((unsigned)(n0 / 128 / kRotGroup) * kRotStep) % (unsigned)n_stage);
    const bf16_t *w = W + (size_t)(n0 + lr) * K + sp * Kp + lq * 8, *x = X + (size_t)min(lr, rows - 1) * ldx + sp * Kp + lq * 8;
    bf16x8 a[kDeep][2], b[kDeep][2];
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int d, int st) {
        const int k = (st + rot < n_stage ? st + rot : st + rot - n_stage) * 64;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            a[d][h] = *reinterpret_cast<const bf16x8 *>(w + k + h * 32);
            b[d][h] = *reinterpret_cast<const bf16x8 *>(x + k + h * 32);
        }
    };
    auto multiply = [&](int d) {
#pragma unroll
        for (int h = 0; h < 2; ++h) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[d][h], b[d][h], acc, 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < kDeep; ++d)
        if (d < n_stage) load(d, d);
    int st = 0;
    for (; st + 2 * kDeep <= n_stage; st += kDeep)
#pragma unroll
        for (int d = 0; d < kDeep; ++d) {
            multiply(d);
            load(d, st + d + kDeep);
        }
    for (; st < n_stage; st += kDeep)
#pragma unroll
        for (int d = 0; d < kDeep; ++d)
            if (st + d < n_stage) {
                multiply(d);
                if (st + d + kDeep < n_stage) load(d, st + d + kDeep);
            }
    planes[sp][lane] = acc;
    __syncthreads();
    if (sp != 0 || lr >= rows) return;
    f32x4 o = planes[0][lane];
#pragma unroll
    for (int s = 1; s < S; ++s) o += planes[s][lane];
    const size_t at = (size_t)lr * N + n0 + 4 * lq;
    if (R) {
        const uint2 rv = *reinterpret_cast<const uint2 *>(R + at);
        o[0] += bf2f(rv.x & 0xffff); o[1] += bf2f(rv.x >> 16);
        o[2] += bf2f(rv.y & 0xffff); o[3] += bf2f(rv.y >> 16);
    }
    uint2 ov;
    ov.x = (uint32_t)f2bf(o[0]) | ((uint32_t)f2bf(o[1]) << 16);
    ov.y = (uint32_t)f2bf(o[2]) | ((uint32_t)f2bf(o[3]) << 16);
    *reinterpret_cast<uint2 *>(Y + at) = ov;
}

// The kernel takes 16 rows, but every workgroup reads all of X for its 16 W rows, so what it costs grows with the rows
// (4096-wide layer, down projection: 1 row 21.6 + 4.1 us of the launch that sums planes -> 23.6, 13 rows 22.0 + 4.2 -> 29.3).
// Whole step, 128-row tiles with planes against this: 2 / 4 / 6 / 8 / 10 / 13 rows 137.3 / 136.4 / 137.0 / 139.0 / 140.0 / 156.2
// -> 130.3 / 132.1 / 133.8 / 137.1 / 139.1 / 157.8 us; a 2048-wide layer's 1 / 4 / 8 / 14 rows 73.3 / 74.3 / 74.6 / 77.7 -> 68.3 /
// 70.7 / 72.9 / 76.8 us.  Past 8 rows the difference is within two runs of one side.
bool gemm_rows16_supported(int rows, int S) { return rows <= 8 && (S == 2 || S == 4 || S == 8); }

hipError_t launch_gemm_rows16(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S) {
#define DYN_ROWS(SC) hipLaunchKernelGGL(gemm_rows16_kernel<SC>, dim3(N / 16), dim3(64 * SC), 0, s, (const bf16_t *)X, ldx, (const bf16_t *)W, \
                                        (const bf16_t *)R, (bf16_t *)Y, rows, N, K)
    if (S == 8) DYN_ROWS(8);
    else if (S == 4) DYN_ROWS(4);
    else DYN_ROWS(2);
#undef DYN_ROWS
    return hipGetLastError();
}

}  // namespace dyn
