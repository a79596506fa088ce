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

// Where the kernel is taken.  Every workgroup reads all of X for its 16 W rows, so what it saves shrinks with the rows, and
// with workgroups that are more than the CUs but do not fill them twice.  Microseconds saved by one projection inside a step
// of one layer / of three (whose weights leave the caches in between), 14 layer widths:
//   at most 256 workgroups, 2 or 4 planes: 1, 4, 8 rows x 2560 x 6912 2.7/3.6, 4.3/2.5, 2.9/2.1, x 3072 x 3072 2.3/3.2, 1.8/2.7, 1.8/2.0,
//     x 4096 x 11008 4.8/4.5, 5.6/5.4, 4.1/5.0, the least x 2048 x 2048 0/1.6, 0.7/1.2, 0.3/0.9
//   at most 256, 8 planes: 1, 4, 6, 8 rows x 4096 x 4096 1.9/1.7, 1.2/2.2, 1.7/2.1, 1.8/1.4, x 4096 x 14336 1.8/1.7, 1.1/0.2, 1.5/0, 0.2/-1.5,
//     x 3072 x 8192 1.5/1.1, 0.5/-0.1, 0.6/0, -0.3/-1.5, x 2048 x 5632 2.0/1.2, 0.8/0.2, 1.6/-0.8, 0.8/-1.2
//   257 to 511: 1, 2, 4 rows x 6144 x 4096 2.7/-0.5, 2.5/-0.5, 0.2/-1.7, x 5120 x 5120 3.4/1.5, 0.6/2.0, 0.5/0.1, x 5120 x 3072 -0.2/-0.1, -0.1/0,
//     -1.2/-0.9, x 4608 x 3584 -0.6/-0.6, -1.6/-1.6, -1.4/-1.1; with long K x 5120 x 13824 0.5/-1.1, -2.0/-1.6, -3.7/-3.5
//   512 and more: three layers, 1, 5, 8 rows x 8192 x 8192 3.2, 2.8, 3.0, x 10240 x 8192 12, 11, 10, x 8192 x 28672 4.5, 2.3, -7.2, x 8192 x 6144
//     1.3, 0.1, -1.5; with 2 planes x 12288 x 4096 -0.3, 0, -1.4
bool gemm_rows16_supported(int rows, int N, int K, int S) {
    if (rows > 8 || (S != 2 && S != 4 && S != 8)) return false;
    const int wg = N / 16;
    if (wg <= 256) return S < 8 || rows <= 6 || (long)rows * K <= 8L * N;
    return wg < 512 ? rows <= 2 && K < 2 * N : S > 2 && rows <= 5;
}

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
