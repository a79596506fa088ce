// Mixture-of-experts pieces around the grouped projections: router, per-expert row lists,
// weighted combine.  Every token's routing and output depend on that token alone, and every
// sum has a fixed order (experts by router rank, split-K planes ascending), so results do
// not depend on how the batch is cut.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "route_row.h"

namespace dyn {

template <typename T, int EM>
__global__ __launch_bounds__(256) void route_kernel(const T *__restrict__ h, int ldh, const float *__restrict__ w_router,
                                                    int32_t *__restrict__ sel, float *__restrict__ wgt, int rows,
                                                    int H, int E, int top_k) {
    __shared__ float part[4][kMaxExperts];
    const int t = blockIdx.x;
    float acc[EM];
#pragma unroll
    for (int e = 0; e < EM; ++e) acc[e] = 0.f;
    for (int k0 = threadIdx.x * 8; k0 < H; k0 += 256 * 8) {
        const bool whole = k0 + 8 <= H;
        float x[8];
        if constexpr (sizeof(T) == 2) {       // one 16-byte load (rows and k0 are 16-byte aligned)
            const u32x4 raw = *reinterpret_cast<const u32x4 *>(h + (size_t)t * ldh + k0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = __uint_as_float(raw[i] << 16);
                x[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = i < 4 || whole ? to_f32<T>(h[(size_t)t * ldh + k0 + i]) : 0.f;
        }
        RouterPiece<EM> p;
        load_piece(p, w_router, H, E, k0);
        add_piece(acc, p, x, E);
    }
    route_choose(acc, part, E, top_k, sel + (size_t)t * top_k, wgt + (size_t)t * top_k);
}

hipError_t launch_route(int dtype, const void *h, int ldh, const float *w_router, int32_t *sel, float *wgt, int rows,
                        int H, int E, int top_k, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
#define DYN_ROUTE(T, EM) hipLaunchKernelGGL((route_kernel<T, EM>), dim3(rows), dim3(256), 0, s, (const T *)h, ldh, w_router, sel, wgt, rows, H, E, top_k)
    if (dtype == 0) {
        if (E <= 8) DYN_ROUTE(float, 8); else DYN_ROUTE(float, 16);
    } else {
        if (E <= 8) DYN_ROUTE(bf16_t, 8); else DYN_ROUTE(bf16_t, 16);
    }
#undef DYN_ROUTE
    return hipGetLastError();
}

// One wave per expert scans the dispatch's pairs, 512 loaded at a time, and appends its own in ascending order.
__global__ void expert_lists_scan_kernel(const int32_t *__restrict__ sel, int n_pairs, int pair_base, int cap, int32_t *__restrict__ counts,
                                         int32_t *__restrict__ lists) {
    const int e = threadIdx.x >> 6, lane = threadIdx.x & 63;
    constexpr int AHEAD = 8;
    int count = 0;
    for (int base = 0; base < n_pairs; base += 64 * AHEAD) {
        int chosen[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int p = base + i * 64 + lane;
            chosen[i] = p < n_pairs ? sel[pair_base + p] : -1;
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const bool mine = chosen[i] == e;
            const unsigned long long mask = __ballot(mine);
            if (mine) lists[(size_t)e * cap + count + __popcll(mask & ((1ull << lane) - 1ull))] = pair_base + base + i * 64 + lane;
            count += __popcll(mask);
        }
    }
    if (lane == 0) counts[e] = count;
}

// More pairs: sixteen waves take consecutive parts of the dispatch's pairs; each counts its part's pairs per expert, the counts of the waves before it
// are its offsets, and every expert's pairs land in ascending order.  Bound by the latency of one load, two barriers and a ballot
// per expert and 64 pairs, twice.
constexpr int kListWaves = 16, kListAhead = 8;             // 64-pair steps of a wave kept in registers between count and store
__global__ __launch_bounds__(kListWaves * 64) void expert_lists_kernel(const int32_t *__restrict__ sel, int n_pairs, int pair_base, int E, int cap,
                                                                       int32_t *__restrict__ counts, int32_t *__restrict__ lists) {
    __shared__ int count[kListWaves][kMaxExperts], before[kMaxExperts];     // this pass's, by wave; those of the passes before
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < kMaxExperts) before[threadIdx.x] = 0;
    constexpr int PASS = kListWaves * 64 * kListAhead;
    for (int base = 0; base < n_pairs; base += PASS) {
        const int steps = (min(PASS, n_pairs - base) + kListWaves * 64 - 1) / (kListWaves * 64), first = base + wave * steps * 64;
        int chosen[kListAhead];
#pragma unroll
        for (int i = 0; i < kListAhead; ++i) {
            const int p = first + i * 64 + lane;
            chosen[i] = i < steps && p < n_pairs ? sel[pair_base + p] : -1;
        }
        for (int e = 0; e < E; ++e) {
            int c = 0;
#pragma unroll
            for (int i = 0; i < kListAhead; ++i)
                if (i < steps) c += __popcll(__ballot(chosen[i] == e));
            if (lane == 0) count[wave][e] = c;
        }
        __syncthreads();
        int at_lane = 0, total = 0;                        // lane e: where this wave's pairs of expert e start; all of this pass's
        if (lane < E) {
            at_lane = before[lane];
#pragma unroll
            for (int w = 0; w < kListWaves; ++w) {
                const int c = count[w][lane];
                at_lane += w < wave ? c : 0;
                total += c;
            }
        }
        for (int e = 0; e < E; ++e) {
            int at = __builtin_amdgcn_readlane(at_lane, e);
#pragma unroll
            for (int i = 0; i < kListAhead; ++i) {
                if (i >= steps) break;
                const bool mine = chosen[i] == e;
                const unsigned long long mask = __ballot(mine);
                if (mine) lists[(size_t)e * cap + at + __popcll(mask & ((1ull << lane) - 1ull))] = pair_base + first + i * 64 + lane;
                at += __popcll(mask);
            }
        }
        __syncthreads();                                   // every wave has read the counts and what came before
        if (wave == 0 && lane < E) before[lane] += total;
    }
    __syncthreads();
    if ((int)threadIdx.x < E) counts[threadIdx.x] = before[threadIdx.x];
}

// The scan takes the time of its steps of 512 pairs, each a load's latency, the sixteen waves that of their ballots, which are as many
// as there are experts (launches inside a layer's steps, scan / sixteen waves, us: 4 experts 520 pairs 3.9 / 3.7, 800 4.6 / 3.8; 8
// experts 700 4.0 / 4.8, 900 4.9 / 5.0, 1000 7.2 / 4.9, 1536 9.7 / 5.6; 16 experts 1040 7.2 / 7.8, 1200 6.4 / 8.0, 1600 8.7 / 8.7, 2048 10.0 /
// 8.8, 3072 15.5 / 10.6).
bool expert_lists_scan(int n_pairs, int E) { return n_pairs <= std::max(512, 100 * E); }

hipError_t launch_expert_lists(const int32_t *sel, int n_pairs, int pair_base, int E, int cap, int32_t *counts,
                               int32_t *lists, hipStream_t s) {
    if (n_pairs <= 0) return hipSuccess;
    if (expert_lists_scan(n_pairs, E)) hipLaunchKernelGGL(expert_lists_scan_kernel, dim3(1), dim3(64 * E), 0, s, sel, n_pairs, pair_base, cap, counts, lists);
    else hipLaunchKernelGGL(expert_lists_kernel, dim3(1), dim3(kListWaves * 64), 0, s, sel, n_pairs, pair_base, E, cap, counts, lists);
    return hipGetLastError();
}

// Four outputs per thread.
template <typename T>
__global__ __launch_bounds__(256) void moe_combine_kernel(const float *__restrict__ planes, size_t plane_stride, int S,
                                                          const float *__restrict__ wgt, const T *__restrict__ x2,
                                                          T *__restrict__ y, size_t n_vec, int H, int top_k) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += (size_t)gridDim.x * 256) {
        const size_t t = i / (H / 4), c = (i % (H / 4)) * 4;
        f32x4 m = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < top_k; ++j) {
            const size_t row = t * top_k + j;
            f32x4 o = *reinterpret_cast<const f32x4 *>(planes + row * H + c);
            for (int p = 1; p < S; ++p) o += *reinterpret_cast<const f32x4 *>(planes + (size_t)p * plane_stride + row * H + c);
            m += o * wgt[row];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) y[t * H + c + r] = from_f32<T>(to_f32<T>(x2[t * H + c + r]) + m[r]);
    }
}

hipError_t launch_moe_combine(int dtype, const float *planes, size_t plane_stride, int S, const float *wgt,
                              const void *x2, void *y, int rows, int H, int top_k, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const size_t n_vec = (size_t)rows * H / 4;
    const int blocks = (int)((n_vec + 255) / 256 < 2048 ? (n_vec + 255) / 256 : 2048);
    if (dtype == 0)
        hipLaunchKernelGGL(moe_combine_kernel<float>, dim3(blocks), dim3(256), 0, s, planes, plane_stride, S, wgt,
                           (const float *)x2, (float *)y, n_vec, H, top_k);
    else
        hipLaunchKernelGGL(moe_combine_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, planes, plane_stride, S, wgt,
                           (const bf16_t *)x2, (bf16_t *)y, n_vec, H, top_k);
    return hipGetLastError();
}

}  // namespace dyn
