// The router's arithmetic for one token, shared by the kernels that apply it.
#pragma once
#include "common.h"
#include "kernels.h"

namespace dyn {

constexpr int kMaxExperts = 16;

// One 256-thread workgroup per token.  Every thread takes contiguous 8-element pieces of the
// row, multiplies them with the same pieces of all E router rows (all loads of a piece are
// independent, so they are in flight together), a butterfly and a fixed-order LDS step add the
// slices, thread 0 picks the top_k largest logits (ties to the lower index) and normalises
// exp(logit - max) over the picked ones.  EM experts at most (a power of two): the butterfly halves
// the experts a lane carries at each of its first steps - lanes that differ in a step's bit keep
// different halves - so 8 experts take 10 shuffles and not 48; every sum pairs the same lanes as a
// butterfly per expert, with the same bits.
template <int N>
__device__ __forceinline__ float halving_sum(const float (&v)[N], int off, int lane) {     // N: experts left, off: the step's lane distance
    if constexpr (N == 1) {
        float x = v[0];
        for (; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
        return x;
    } else {
        const bool up = lane & off;
        float keep[N / 2];
#pragma unroll
        for (int e = 0; e < N / 2; ++e) {
            const float give = up ? v[e] : v[e + N / 2], mine = up ? v[e + N / 2] : v[e];
            keep[e] = mine + __shfl_xor(give, off, 64);
        }
        return halving_sum<N / 2>(keep, off >> 1, lane);
    }
}

// The part of the logits that a thread's eight elements from k0 on give, in ascending order.
template <int EM>
struct RouterPiece { f32x4 w[EM][2]; };
template <int EM>
__device__ __forceinline__ void load_piece(RouterPiece<EM> &p, const float *__restrict__ w_router, int H, int E, int k0) {
    const bool whole = k0 + 8 <= H;                    // fp32 rows may end in a half piece (H is a multiple of 4)
#pragma unroll
    for (int e = 0; e < EM; ++e)
        if (e < E) {
            p.w[e][0] = *reinterpret_cast<const f32x4 *>(w_router + (size_t)e * H + k0);
            p.w[e][1] = whole ? *reinterpret_cast<const f32x4 *>(w_router + (size_t)e * H + k0 + 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
}
template <int EM>
__device__ __forceinline__ void add_piece(float (&acc)[EM], const RouterPiece<EM> &p, const float (&x)[8], int E) {
#pragma unroll
    for (int e = 0; e < EM; ++e)
        if (e < E) {
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[e] = fmaf(x[i], p.w[e][i >> 2][i & 3], acc[e]);
        }
}

// The logits of a row whose vectors of eight a thread normalises, vector i = tid + n * 256 as k0 = 8 i: the first two vectors' router elements are
// loaded before the norm is known (load()), the others when their turn comes.
template <int EM>
struct RowRouter {
    RouterPiece<EM> ahead[2];
    float acc[EM];
    const GemmRoute &r;
    int H;
    __device__ __forceinline__ RowRouter(const GemmRoute &route, int width) : r(route), H(width) {
#pragma unroll
        for (int e = 0; e < EM; ++e) acc[e] = 0.f;
    }
    __device__ __forceinline__ void load() {
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int k0 = ((int)threadIdx.x + n * 256) * 8;
            if (k0 < H) load_piece(ahead[n], r.w_router, H, r.E, k0);
        }
    }
    template <typename V>
    __device__ __forceinline__ void operator()(int i, const V &o) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = bf2f(o[e]);
        if (i < 256) add_piece(acc, ahead[0], x, r.E);
        else if (i < 512) add_piece(acc, ahead[1], x, r.E);
        else {
            RouterPiece<EM> p;
            load_piece(p, r.w_router, H, r.E, i * 8);
            add_piece(acc, p, x, r.E);
        }
    }
};

// The token's choice from its 256 threads' slices; part: LDS of its own.  Every thread of the workgroup calls this (it synchronises).
template <int EM>
__device__ __forceinline__ void route_choose(const float (&acc)[EM], float (*part)[kMaxExperts], int E, int top_k, int32_t *__restrict__ sel,
                                             float *__restrict__ wgt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        const float v = halving_sum<EM>(acc, 32, lane);
        // lane bits 5, 4, .. (one per halving) name the expert, high bit first: the lanes below them all hold its sum
        constexpr int PER = 64 / EM;
        if (lane % PER == 0) part[wave][lane / PER] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    float logit[EM], ex[EM];
    int pick[EM];
#pragma unroll
    for (int e = 0; e < EM; ++e) logit[e] = ((part[0][e] + part[1][e]) + part[2][e]) + part[3][e];
    // No array is indexed with a run-time value here: that would move it from registers to scratch
    // memory, and this single thread's dependent accesses to it were most of the kernel's time.
    unsigned used = 0;
    float mx = 0.f, denom = 0.f;
#pragma unroll
    for (int j = 0; j < EM; ++j)
        if (j < top_k) {
            int best = -1;
            float best_val = 0.f;
#pragma unroll
            for (int e = 0; e < EM; ++e)
                if (e < E && !((used >> e) & 1u) && (best < 0 || logit[e] > best_val)) { best = e; best_val = logit[e]; }
            used |= 1u << best;
            if (j == 0) mx = best_val;        // picks come in descending order: the first is the maximum
            ex[j] = expf(best_val - mx);
            pick[j] = best;
            denom += ex[j];
        }
#pragma unroll
    for (int j = 0; j < EM; ++j)
        if (j < top_k) { sel[j] = pick[j]; wgt[j] = ex[j] / denom; }
}

}  // namespace dyn
