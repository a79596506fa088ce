// RMSNorm of one row by 256 threads, shared by the kernels that run it.
#pragma once
#include "common.h"

namespace dyn {

// out = x * g / sqrt(mean(x^2) + eps); tid: 0..255 within the row's threads, part: 4 floats of LDS of their own.
// The row and the gains are loaded together, once: with few rows the launch is one workgroup's latency
// long.  Every thread of the workgroup calls this (it synchronises); live = false computes nothing.  each(i, o) is given the vectors stored.
struct NoVector { template <typename V> __device__ __forceinline__ void operator()(int, const V &) const {} };
template <typename T, typename F = NoVector>
__device__ __forceinline__ void rmsnorm_row(const T *__restrict__ x, const T *__restrict__ g, T *__restrict__ out, int H, float eps, int tid,
                                            float *part, bool live, F &&each = F()) {
    constexpr int V = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(V)));
    const vec_t *xr = reinterpret_cast<const vec_t *>(x), *gr = reinterpret_cast<const vec_t *>(g);
    vec_t *orow = reinterpret_cast<vec_t *>(out);
    const int nv = live ? H / V : 0;
    constexpr int KEEP = 4;                    // vectors of the row and of g a thread keeps in registers; beyond, both are read (again)
    vec_t kept[KEEP], gain[KEEP];
#pragma unroll
    for (int n = 0; n < KEEP; ++n) {
        const int i = tid + n * 256;
        if (i < nv) { kept[n] = xr[i]; gain[n] = gr[i]; }
    }
    float ss = 0.f;
    auto square = [&](const vec_t &v) {
#pragma unroll
        for (int e = 0; e < V; ++e) { const float f = to_f32<T>(v[e]); ss = __builtin_fmaf(f, f, ss); }
    };
#pragma unroll
    for (int n = 0; n < KEEP; ++n)
        if (tid + n * 256 < nv) square(kept[n]);
    for (int i = tid + KEEP * 256; i < nv; i += 256) square(xr[i]);
    ss = wave_sum(ss);
    if ((tid & 63) == 0) part[tid >> 6] = ss;
    __syncthreads();
    const float total = ((part[0] + part[1]) + part[2]) + part[3];
    const float r = 1.0f / sqrtf(total / (float)H + eps);
    auto scaled = [&](const vec_t &v, const vec_t &gv) {
        vec_t o;
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = from_f32<T>(to_f32<T>(v[e]) * r * to_f32<T>(gv[e]));
        return o;
    };
#pragma unroll
    for (int n = 0; n < KEEP; ++n)
        if (tid + n * 256 < nv) {
            const vec_t o = scaled(kept[n], gain[n]);
            orow[tid + n * 256] = o;
            each(tid + n * 256, o);
        }
    for (int i = tid + KEEP * 256; i < nv; i += 256) {
        const vec_t o = scaled(xr[i], gr[i]);
        orow[i] = o;
        each(i, o);
    }
}

}  // namespace dyn
