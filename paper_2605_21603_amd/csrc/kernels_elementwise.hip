// RMSNorm, rotary + KV-cache append, SiLU-gate: the memory-bound elementwise operators of
// the layer (the paper's "normalization" class, Section 2).  fp32 arithmetic, storage
// type T.  Every output row depends on its own input row only and is reduced in an order
// fixed by the block shape, so results do not depend on how a batch is split.
#include "common.h"
#include "kernels.h"
#include "norm_row.h"
#include "rotary.h"
#include "route_row.h"

namespace dyn {

// ------------------------------------------------------------------ RMSNorm
// One 256-thread workgroup per row (norm_row.h).
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const T *__restrict__ x, const T *__restrict__ g,
                                                      T *__restrict__ out, int ld_out, int H, float eps) {
    __shared__ float part[4];
    const size_t row = blockIdx.x;
    rmsnorm_row<T>(x + row * H, g, out + row * ld_out, H, eps, threadIdx.x, part, true);
}

// The same with the router behind it: a launch of its own reads the row again, and the router's weights behind the norm rather than beside it.
// Latency bounds it: one row, the router's elements from the L2, two sums over the workgroup, one thread's choice.  (Hidden 4096, 8 experts, one
// row: norm 4.6 + router 11.7 -> 8.8 us, the step 238.7 -> 233.1; 256 rows with 8 planes 10.2 + 12.3 -> 16.0 us, the step 861 -> 859.)
__global__ __launch_bounds__(256) void rmsnorm_route_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ g, bf16_t *__restrict__ out,
                                                            int ld_out, int H, float eps, GemmRoute route) {
    __shared__ float part[4], slices[4][kMaxExperts];
    const size_t row = blockIdx.x;
    RowRouter<8> router(route, H);
    router.load();
    rmsnorm_row<bf16_t, RowRouter<8> &>(x + row * H, g, out + row * ld_out, H, eps, threadIdx.x, part, true, router);
    route_choose<8>(router.acc, slices, route.E, route.top_k, route.sel + row * route.top_k, route.wgt + row * route.top_k);
}

// Rows up to which the router joins the norm: the router's elements in registers leave a CU two such workgroups, and more rows than these take
// hold at once take longer than two launches (1120 rows: 6.8 + 13.0 us apart, 21.4 together).
constexpr int kNormRouteRows = 512;
static hipError_t route_rows(const GemmRoute &to, const void *h, int ld_h, int rows, int H, hipStream_t s) {
    return launch_route(1, h, ld_h, to.w_router, to.sel, to.wgt, rows, H, to.E, to.top_k, s);
}

hipError_t launch_rmsnorm(int dtype, const void *x, const void *g, void *out, int ld_out, int rows, int H, float eps,
                          hipStream_t s, const GemmRoute *route) {
    if (rows <= 0) return hipSuccess;
    if (route && route->w_router && rows > kNormRouteRows) {
        const hipError_t e = launch_rmsnorm(dtype, x, g, out, ld_out, rows, H, eps, s);
        return e == hipSuccess ? route_rows(*route, out, ld_out, rows, H, s) : e;
    }
    if (route && route->w_router) {
        hipLaunchKernelGGL(rmsnorm_route_kernel, dim3(rows), dim3(256), 0, s, (const bf16_t *)x, (const bf16_t *)g, (bf16_t *)out, ld_out, H, eps, *route);
        return hipGetLastError();
    }
    if (dtype == 0)
        hipLaunchKernelGGL(rmsnorm_kernel<float>, dim3(rows), dim3(256), 0, s, (const float *)x, (const float *)g,
                           (float *)out, ld_out, H, eps);
    else
        hipLaunchKernelGGL(rmsnorm_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, (const bf16_t *)x,
                           (const bf16_t *)g, (bf16_t *)out, ld_out, H, eps);
    return hipGetLastError();
}

// Split-K reduce of a projection fused with the RMSNorm that follows it (bf16): one 256-thread
// workgroup per row sums the row's S fp32 planes in plane order, adds the residual, rounds to
// bf16 (the projection's output Y), and normalises the rounded values exactly as rmsnorm_kernel
// does - same thread-to-column mapping, same order of the sum of squares - so a row has the same
// bits as with gemm_reduce_kernel followed by rmsnorm_kernel.
// (SC = the split factor as a compile-time constant, so that a row's plane loads are all issued
// before the first is added - one workgroup per row has nothing else to hide their latency with;
// 0 = any factor, loop.)
// ROUTE: the router behind the norm, as rmsnorm_route_kernel applies it.
template <int SC, bool ROUTE>
__global__ __launch_bounds__(256) void gemm_reduce_norm_kernel(const float *__restrict__ P, size_t plane_stride, int S,
                                                               const bf16_t *__restrict__ R, bf16_t *__restrict__ Y,
                                                               const bf16_t *__restrict__ g, bf16_t *__restrict__ out,
                                                               int ld_out, int H, float eps, GemmRoute route) {
    typedef bf16_t vec_t __attribute__((ext_vector_type(8)));
    RowRouter<ROUTE ? 8 : 1> router(route, H);
    constexpr int KEEP = 4;                                 // vectors a thread keeps in registers (H <= 8192); beyond, Y is read back
    const size_t row = blockIdx.x;
    const int nv = H / 8;
    vec_t kept[KEEP];
    // f(i, n) for the thread's vectors i, n counting them.  With the router behind the norm the compiler does not unroll a loop over them, and kept[n] would
    // lie in scratch memory (80 bytes a lane, 231 registers -> 179): there n is a constant, KEEP for all beyond.
    auto vectors = [&](auto &&f) {
        if constexpr (ROUTE) {
            static_for<0, KEEP>([&](auto n) {
                if ((int)threadIdx.x + n * 256 < nv) f((int)threadIdx.x + n * 256, n);
            });
            for (int i = (int)threadIdx.x + KEEP * 256; i < nv; i += 256) f(i, std::integral_constant<int, KEEP>());
        } else {
            int n = 0;
            for (int i = threadIdx.x; i < nv; i += 256, ++n) f(i, n);
        }
    };
    float ss = 0.f;
    vectors([&](int i, auto n) {
        const float *p = P + row * H + (size_t)i * 8;
        f32x4 a, b;
        vec_t rv{};
        if (R) rv = *reinterpret_cast<const vec_t *>(R + row * H + (size_t)i * 8);
        if constexpr (SC > 0) {
            f32x4 pa[SC], pb[SC];
#pragma unroll
            for (int sp = 0; sp < SC; ++sp) {
                pa[sp] = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride);
                pb[sp] = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride + 4);
            }
            a = pa[0];
            b = pb[0];
#pragma unroll
            for (int sp = 1; sp < SC; ++sp) {
                a[0] += pa[sp][0]; a[1] += pa[sp][1]; a[2] += pa[sp][2]; a[3] += pa[sp][3];
                b[0] += pb[sp][0]; b[1] += pb[sp][1]; b[2] += pb[sp][2]; b[3] += pb[sp][3];
            }
        } else {
            a = *reinterpret_cast<const f32x4 *>(p);
            b = *reinterpret_cast<const f32x4 *>(p + 4);
            for (int sp = 1; sp < S; ++sp) {
                const f32x4 c = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride);
                const f32x4 d = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride + 4);
                a[0] += c[0]; a[1] += c[1]; a[2] += c[2]; a[3] += c[3];
                b[0] += d[0]; b[1] += d[1]; b[2] += d[2]; b[3] += d[3];
            }
        }
        if (R) {
            a[0] += bf2f(rv[0]); a[1] += bf2f(rv[1]); a[2] += bf2f(rv[2]); a[3] += bf2f(rv[3]);
            b[0] += bf2f(rv[4]); b[1] += bf2f(rv[5]); b[2] += bf2f(rv[6]); b[3] += bf2f(rv[7]);
        }
        vec_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = f2bf(a[e]); v[e + 4] = f2bf(b[e]); }
        *reinterpret_cast<vec_t *>(Y + row * H + (size_t)i * 8) = v;
        if (n < KEEP) kept[n < KEEP ? n : 0] = v;
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float f = bf2f(v[e]); ss = __builtin_fmaf(f, f, ss); }
    });
    if constexpr (ROUTE) router.load();                     // beside the row's sum
    ss = wave_sum(ss);
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float total = ((part[0] + part[1]) + part[2]) + part[3];
    const float r = 1.0f / sqrtf(total / (float)H + eps);
    vectors([&](int i, auto n) {
        // beyond the kept vectors a thread reads back what it stored itself
        const vec_t v = n < KEEP ? kept[n < KEEP ? n : 0] : *reinterpret_cast<const vec_t *>(Y + row * H + (size_t)i * 8);
        const vec_t gv = *reinterpret_cast<const vec_t *>(g + (size_t)i * 8);
        vec_t o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = f2bf(bf2f(v[e]) * r * bf2f(gv[e]));
        *reinterpret_cast<vec_t *>(out + row * ld_out + (size_t)i * 8) = o;
        if constexpr (ROUTE) router(i, o);
    });
    if constexpr (ROUTE) {
        __shared__ float slices[4][kMaxExperts];
        route_choose<8>(router.acc, slices, route.E, route.top_k, route.sel + row * route.top_k, route.wgt + row * route.top_k);
    }
}

hipError_t launch_reduce_norm(const float *P, size_t plane_stride, int S, const void *R, void *Y, const void *g, void *out,
                              int ld_out, int rows, int H, float eps, hipStream_t s, const GemmRoute *route) {
    if (rows <= 0) return hipSuccess;
    if (route && route->w_router && rows > kNormRouteRows) {
        const hipError_t e = launch_reduce_norm(P, plane_stride, S, R, Y, g, out, ld_out, rows, H, eps, s);
        return e == hipSuccess ? route_rows(*route, out, ld_out, rows, H, s) : e;
    }
    const GemmRoute none, &to = route ? *route : none;
#define DYN_RN_OF(SC, ROUTE) hipLaunchKernelGGL((gemm_reduce_norm_kernel<SC, ROUTE>), dim3(rows), dim3(256), 0, s, P, plane_stride, S, (const bf16_t *)R, \
                                                (bf16_t *)Y, (const bf16_t *)g, (bf16_t *)out, ld_out, H, eps, to)
#define DYN_RN(SC) if (to.w_router) DYN_RN_OF(SC, true); else DYN_RN_OF(SC, false)
    switch (S) {
        case 2: DYN_RN(2); break;
        case 4: DYN_RN(4); break;
        case 8: DYN_RN(8); break;
        default: DYN_RN(0); break;
    }
#undef DYN_RN
#undef DYN_RN_OF
    return hipGetLastError();
}

// ------------------------------------------------------------------ rotary + cache append
// One thread per (token, head, pair index i < d/2); heads are the q heads, then the k heads,
// then the v heads (a v "pair" is just two elements to copy).  The angle pos * theta_i is
// formed and reduced to [-pi, pi] in fp64, then sine and cosine are taken in fp32, so the
// rotation is good to fp32 rounding at any position.
template <typename T>
__global__ __launch_bounds__(256) void rope_kv_kernel(T *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                      const int32_t *__restrict__ pos_of_token,
                                                      const int32_t *__restrict__ block_table,
                                                      T *__restrict__ k_cache, T *__restrict__ v_cache,
                                                      RopeTable tab, AttnShape sh) {
    const int t = blockIdx.x;
    const int d = sh.head_dim, half = d >> 1;
    const int item = blockIdx.y * 256 + threadIdx.x;
    const int hh = item / half, i = item % half;
    if (hh >= sh.n_q + 2 * sh.n_kv) return;
    const int pos = pos_of_token[t];
    T *z = qkv + (size_t)t * ((sh.n_q + 2 * sh.n_kv) * d) + hh * d;
    const float a = to_f32<T>(z[i]), b = to_f32<T>(z[i + half]);
    if (hh >= sh.n_q + sh.n_kv) {                        // v head -> V page [kvh][d][slot]
        const int g = hh - sh.n_q - sh.n_kv;
        const int page = block_table[(size_t)seq_of_token[t] * sh.max_pages_per_seq + pos / sh.page_size];
        T *vp = v_cache + ((size_t)page * sh.n_kv + g) * d * sh.page_size + pos % sh.page_size;
        vp[(size_t)i * sh.page_size] = z[i];
        vp[(size_t)(i + half) * sh.page_size] = z[i + half];
        return;
    }
    float s, c;
    rotary_angle(pos, tab.inv_freq[i], s, c);
    const T lo = from_f32<T>(rotated_lo(a, b, c, s)), hi = from_f32<T>(rotated_hi(a, b, c, s));
    if (hh < sh.n_q) {                                   // q head, in place
        z[i] = lo;
        z[i + half] = hi;
    } else {                                             // k head -> K page [kvh][slot][d]
        const int g = hh - sh.n_q;
        const int page = block_table[(size_t)seq_of_token[t] * sh.max_pages_per_seq + pos / sh.page_size];
        T *kp = k_cache + (((size_t)page * sh.n_kv + g) * sh.page_size + pos % sh.page_size) * d;
        kp[i] = lo;
        kp[i + half] = hi;
    }
}

// Vector form for head dims whose half is a multiple of the 16-byte vector: one workgroup per
// token.  The d/2 angles of the token are reduced and their sine / cosine taken once (not once
// per head) into LDS; then a thread rotates V pair indices of one head with 16-byte loads and
// stores (q in place, k into its cache page), and the v heads are scattered into the
// position-fastest V page element by element.  Same arithmetic per element as the scalar form.
// Many rows (RUNS): 16 rows of one sequence at consecutive positions from a multiple of 16 on - a run, wherever in the launch
// it starts - share a page of whole 16s, where a column's 16 positions are adjacent and leave as whole 16-byte stores, 256
// columns a workgroup, a column a thread.  A row of no run is its own workgroup's, two bytes to each of its columns' 32.
// A prompt is runs but for its ends whatever row and position it starts at (launch, 32 + 16 heads of 128, bf16, a workgroup per row -> by
// runs: 2048 rows 17.4 -> 12.9 us, behind 1001 positions 17.6 -> 14.2, behind three single tokens' rows 18.5 -> 13.4, prompts of 511 + 1000 +
// 600 19.2 -> 14.8; fp32, 16 + 8 heads of 64: 2048 behind 1001 8.9 -> 7.0).
struct RunWindow {                             // of rows base .. base + 30, one a lane
    int row, pos, seq;
    bool in;
    __device__ __forceinline__ RunWindow(const int32_t *__restrict__ seq_of_token, const int32_t *__restrict__ pos_of_token, int base, int rows) {
        const int lane = threadIdx.x & 63;
        row = base + lane;
        in = lane < 31 && row >= 0 && row < rows;
        pos = pos_of_token[in ? row : 0];
        seq = seq_of_token[in ? row : 0];
    }
    // Which of the first 16 rows a run starts at, a bit each: at most one.  Every lane of the wave takes part.
    __device__ __forceinline__ unsigned starts() const {
        const int lane = threadIdx.x & 63, seq_before = __shfl_up(seq, 1, 64), pos_before = __shfl_up(pos, 1, 64);
        const unsigned long long follows = __ballot(lane > 0 && in && row > 0 && seq == seq_before && pos == pos_before + 1);
        return (unsigned)__ballot(lane < 16 && in && pos % 16 == 0 && (follows >> (lane + 1) & 0x7fff) == 0x7fff);
    }
};

// The run that starts in rows t0 .. t0 + 15, column c of the v heads.
template <typename T>
__device__ __forceinline__ void append_v_run(const T *__restrict__ qkv, const int32_t *__restrict__ seq_of_token, const int32_t *__restrict__ pos_of_token,
                                             const int32_t *__restrict__ block_table, T *__restrict__ v_cache, const AttnShape &sh, int t0, int c, int rows) {
    constexpr int V = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(V)));
    const RunWindow window(seq_of_token, pos_of_token, t0, rows);
    const unsigned starts = window.starts();
    if (!starts || c >= sh.n_kv * sh.head_dim) return;
    const int first = __builtin_ctz(starts), d = sh.head_dim, width = (sh.n_q + 2 * sh.n_kv) * d, g = c / d, i = c % d;
    const int pos = __builtin_amdgcn_readlane(window.pos, first), seq = __builtin_amdgcn_readlane(window.seq, first);
    const T *const v0 = qkv + (size_t)(t0 + first) * width + (size_t)(sh.n_q + sh.n_kv) * d + c;
    T v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = v0[(size_t)k * width];
    const int page = block_table[(size_t)seq * sh.max_pages_per_seq + pos / sh.page_size];
    T *const vp = v_cache + (((size_t)page * sh.n_kv + g) * d + i) * sh.page_size + pos % sh.page_size;
#pragma unroll
    for (int k = 0; k < 16; k += V) {
        vec_t o;
#pragma unroll
        for (int j = 0; j < V; ++j) o[j] = v[k + j];
        *reinterpret_cast<vec_t *>(vp + k) = o;
    }
}

template <typename T, bool RUNS, int AHEAD>
__global__ __launch_bounds__(256) void rope_kv_vec_kernel(T *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                          const int32_t *__restrict__ pos_of_token,
                                                          const int32_t *__restrict__ block_table,
                                                          T *__restrict__ k_cache, T *__restrict__ v_cache,
                                                          RopeTable tab, AttnShape sh, int rows) {
    constexpr int V = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(V)));
    __shared__ float cs[2][128];                          // cos, sin of the token's angles (head_dim <= 256)
    const int v_across = (sh.n_kv * sh.head_dim + 255) / 256, v_groups = RUNS ? (rows + 15) / 16 * v_across : 0;
    if (RUNS && (int)blockIdx.x < v_groups) {
        append_v_run<T>(qkv, seq_of_token, pos_of_token, block_table, v_cache, sh, (int)blockIdx.x / v_across * 16,
                        (int)blockIdx.x % v_across * 256 + (int)threadIdx.x, rows);
        return;
    }
    const int t = blockIdx.x - v_groups;
    const int d = sh.head_dim, half = d >> 1;
    T *row = qkv + (size_t)t * ((sh.n_q + 2 * sh.n_kv) * d);
    const int per_head = half / V, n_rot = (sh.n_q + sh.n_kv) * per_head;
    // a token's units are dealt over gridDim.y workgroups (few tokens: more workgroups than tokens); a thread's first AHEAD are
    // loaded ahead of the position, the angles and the barrier behind them
    const int first = blockIdx.y * 256 + threadIdx.x, step = gridDim.y * 256;
    vec_t a[AHEAD > 0 ? AHEAD : 1], b[AHEAD > 0 ? AHEAD : 1];
    auto load = [&](int u, vec_t &lo, vec_t &hi) {
        const T *z = row + u / per_head * d + u % per_head * V;
        lo = *reinterpret_cast<const vec_t *>(z);
        hi = *reinterpret_cast<const vec_t *>(z + half);
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j)
        if (first + j * step < n_rot) load(first + j * step, a[j], b[j]);
    const RunWindow window(seq_of_token, pos_of_token, RUNS ? t - 15 : t, rows);      // a run that holds row t starts in its first 16
    const int pos = pos_of_token[t];
    for (int i = threadIdx.x; i < half; i += 256) {
        float sn, c;
        rotary_angle(pos, tab.inv_freq[i], sn, c);
        cs[0][i] = c;
        cs[1][i] = sn;
    }
    const int page = block_table[(size_t)seq_of_token[t] * sh.max_pages_per_seq + pos / sh.page_size];
    const int slot = pos % sh.page_size;
    __syncthreads();
    auto rotate = [&](int u, const vec_t &va, const vec_t &vb) {
        const int hh = u / per_head, i0 = (u % per_head) * V;
        vec_t lo, hi;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float c = cs[0][i0 + e], sn = cs[1][i0 + e], fa = to_f32<T>(va[e]), fb = to_f32<T>(vb[e]);
            lo[e] = from_f32<T>(rotated_lo(fa, fb, c, sn));
            hi[e] = from_f32<T>(rotated_hi(fa, fb, c, sn));
        }
        T *dst = hh < sh.n_q ? row + hh * d : k_cache + (((size_t)page * sh.n_kv + (hh - sh.n_q)) * sh.page_size + slot) * d;
        *reinterpret_cast<vec_t *>(dst + i0) = lo;
        *reinterpret_cast<vec_t *>(dst + i0 + half) = hi;
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j)
        if (first + j * step < n_rot) rotate(first + j * step, a[j], b[j]);
    for (int u = first + AHEAD * step; u < n_rot; u += step) {
        load(u, a[0], b[0]);
        rotate(u, a[0], b[0]);
    }
    if (RUNS && window.starts()) return;
    const T *vrow = row + (sh.n_q + sh.n_kv) * d;
    for (int u = first; u < sh.n_kv * d; u += step) {                   // v heads -> V page [kvh][d][slot]
        const int g = u / d, i = u % d;
        v_cache[(((size_t)page * sh.n_kv + g) * d + i) * sh.page_size + slot] = vrow[u];
    }
}

// Split-K reduce of the qkv projection fused with rotary + cache append (bf16, the vector form's
// shapes): the a / b halves of a rotation unit are the sums of the S fp32 planes in plane order,
// rounded to bf16 - the values gemm_reduce_kernel would have stored - and from there on the
// arithmetic of rope_kv_vec_kernel, unit for unit.  q' goes to the qkv row, k' and v to the cache
// pages; the unrotated k and v are not stored anywhere (nothing reads them).
template <int SC>
__global__ __launch_bounds__(256) void gemm_reduce_rope_kernel(const float *__restrict__ P, size_t plane_stride, int S,
                                                               bf16_t *__restrict__ qkv, const int32_t *__restrict__ seq_of_token,
                                                               const int32_t *__restrict__ pos_of_token,
                                                               const int32_t *__restrict__ block_table,
                                                               bf16_t *__restrict__ k_cache, bf16_t *__restrict__ v_cache,
                                                               RopeTable tab, AttnShape sh) {
    typedef bf16_t vec_t __attribute__((ext_vector_type(8)));
    constexpr int V = 8;
    __shared__ float cs[2][128];
    const int t = blockIdx.x;
    const int d = sh.head_dim, half = d >> 1;
    const int width = (sh.n_q + 2 * sh.n_kv) * d, vbase = (sh.n_q + sh.n_kv) * d;
    const float *prow = P + (size_t)t * width;
    bf16_t *row = qkv + (size_t)t * width;
    auto summed = [&](int col) {                           // eight consecutive columns of the row, planes added in order, rounded
        const float *p = prow + col;
        f32x4 a, b;
        if constexpr (SC > 0) {                            // all plane loads in flight before the first add
            f32x4 pa[SC], pb[SC];
#pragma unroll
            for (int sp = 0; sp < SC; ++sp) {
                pa[sp] = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride);
                pb[sp] = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride + 4);
            }
            a = pa[0];
            b = pb[0];
#pragma unroll
            for (int sp = 1; sp < SC; ++sp) {
                a[0] += pa[sp][0]; a[1] += pa[sp][1]; a[2] += pa[sp][2]; a[3] += pa[sp][3];
                b[0] += pb[sp][0]; b[1] += pb[sp][1]; b[2] += pb[sp][2]; b[3] += pb[sp][3];
            }
        } else {
            a = *reinterpret_cast<const f32x4 *>(p);
            b = *reinterpret_cast<const f32x4 *>(p + 4);
            for (int sp = 1; sp < S; ++sp) {
                const f32x4 c = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride);
                const f32x4 e = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride + 4);
                a[0] += c[0]; a[1] += c[1]; a[2] += c[2]; a[3] += c[3];
                b[0] += e[0]; b[1] += e[1]; b[2] += e[2]; b[3] += e[3];
            }
        }
        vec_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = f2bf(a[e]); v[e + 4] = f2bf(b[e]); }
        return v;
    };
    // units: rotations of eight pairs of a q or k head, then eight head-dim indices of a v head.  A thread's first
    // unit is summed before the angles are taken: the planes arrive beside the position, its page and the sines.
    const int per_head = half / V, n_rot = (sh.n_q + sh.n_kv) * per_head, n_units = n_rot + sh.n_kv * d / V;
    const int first = blockIdx.y * 256 + threadIdx.x, step = gridDim.y * 256;
    auto sum_unit = [&](int u, vec_t &a, vec_t &b) {
        if (u < n_rot) {
            const int col = (u / per_head) * d + (u % per_head) * V;
            a = summed(col);
            b = summed(col + half);
        } else if (u < n_units) {
            a = summed(vbase + (u - n_rot) * V);
        }
    };
    vec_t a, b;
    sum_unit(first, a, b);
    const int pos = pos_of_token[t];
    const int page = block_table[(size_t)seq_of_token[t] * sh.max_pages_per_seq + pos / sh.page_size];
    const int slot = pos % sh.page_size;
    for (int i = threadIdx.x; i < half; i += 256) {
        float sn, c;
        rotary_angle(pos, tab.inv_freq[i], sn, c);
        cs[0][i] = c;
        cs[1][i] = sn;
    }
    __syncthreads();
    for (int u = first; u < n_units; u += step) {
        if (u != first) sum_unit(u, a, b);
        if (u < n_rot) {
            const int hh = u / per_head, i0 = (u % per_head) * V;
            vec_t lo, hi;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float c = cs[0][i0 + e], sn = cs[1][i0 + e], fa = bf2f(a[e]), fb = bf2f(b[e]);
                lo[e] = f2bf(rotated_lo(fa, fb, c, sn));
                hi[e] = f2bf(rotated_hi(fa, fb, c, sn));
            }
            bf16_t *dst = hh < sh.n_q ? row + hh * d : k_cache + (((size_t)page * sh.n_kv + (hh - sh.n_q)) * sh.page_size + slot) * d;
            *reinterpret_cast<vec_t *>(dst + i0) = lo;
            *reinterpret_cast<vec_t *>(dst + i0 + half) = hi;
        } else {                                                       // v head -> V page [kvh][d][slot]
            const int g = ((u - n_rot) * V) / d, i = ((u - n_rot) * V) % d;
            bf16_t *vp = v_cache + (((size_t)page * sh.n_kv + g) * d + i) * sh.page_size + slot;
#pragma unroll
            for (int e = 0; e < V; ++e) vp[(size_t)e * sh.page_size] = a[e];
        }
    }
}

bool reduce_rope_supported(int dtype, const AttnShape &sh) { return dtype == 1 && (sh.head_dim / 2) % 8 == 0 && sh.head_dim <= 256; }

hipError_t launch_reduce_rope(const float *P, size_t plane_stride, int S, void *qkv, const int32_t *seq_of_token,
                              const int32_t *pos_of_token, const int32_t *block_table, void *k_cache, void *v_cache,
                              const RopeTable &tab, const AttnShape &sh, int rows, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    // a token's units over as many workgroups as give every thread one when tokens are few
    const int units = (sh.n_q + sh.n_kv) * (sh.head_dim / 16) + sh.n_kv * sh.head_dim / 8;
    const dim3 grid(rows, rows < 512 ? (units + 255) / 256 : 1);
#define DYN_RR(SC) hipLaunchKernelGGL(gemm_reduce_rope_kernel<SC>, grid, dim3(256), 0, s, P, plane_stride, S, (bf16_t *)qkv, seq_of_token, \
                                      pos_of_token, block_table, (bf16_t *)k_cache, (bf16_t *)v_cache, tab, sh)
    switch (S) {
        case 2: DYN_RR(2); break;
        case 4: DYN_RR(4); break;
        case 8: DYN_RR(8); break;
        default: DYN_RR(0); break;
    }
#undef DYN_RR
    return hipGetLastError();
}

hipError_t launch_rope_kv(int dtype, void *qkv, const int32_t *seq_of_token, const int32_t *pos_of_token,
                          const int32_t *block_table, void *k_cache, void *v_cache, const RopeTable &tab,
                          const AttnShape &sh, int rows, int long_rows, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int vec = dtype == 0 ? 4 : 8;
    if ((sh.head_dim / 2) % vec == 0 && sh.head_dim <= 256) {
        // From 512 rows on there are workgroups enough with one per row.  The v heads go by runs where pages hold whole ones and a
        // quarter of the rows may belong to some: looking for runs where there are none costs up to a microsecond (1100 single tokens: bf16
        // 20.2 us by rows, 21.1 by runs, fp32 8.9, 9.2), and a row in a run saves 2 ns.  By rows nothing is loaded ahead (two units: 21.2, 9.3).
        const bool runs = long_rows >= rows / 4 && sh.page_size % 16 == 0 && ((uintptr_t)v_cache & 15) == 0;
        const int run_groups = (rows + 15) / 16 * ((sh.n_kv * sh.head_dim + 255) / 256);
#define DYN_ROPE(T, RUNS, AHEAD, GRID)                                                                                                          \
    hipLaunchKernelGGL((rope_kv_vec_kernel<T, RUNS, AHEAD>), GRID, dim3(256), 0, s, (T *)qkv, seq_of_token, pos_of_token, block_table, (T *)k_cache, \
                       (T *)v_cache, tab, sh, rows)
        if (rows >= 512 && runs) {
            if (dtype == 0) DYN_ROPE(float, true, 2, dim3(rows + run_groups)); else DYN_ROPE(bf16_t, true, 2, dim3(rows + run_groups));
        } else if (rows >= 512) {
            if (dtype == 0) DYN_ROPE(float, false, 0, dim3(rows)); else DYN_ROPE(bf16_t, false, 0, dim3(rows));
        } else {
            if (dtype == 0) DYN_ROPE(float, false, 2, dim3(rows, 4)); else DYN_ROPE(bf16_t, false, 2, dim3(rows, 4));
        }
#undef DYN_ROPE
        return hipGetLastError();
    }
    const int items = (sh.n_q + 2 * sh.n_kv) * (sh.head_dim / 2);
    const dim3 grid(rows, (items + 255) / 256);
    if (dtype == 0)
        hipLaunchKernelGGL(rope_kv_kernel<float>, grid, dim3(256), 0, s, (float *)qkv, seq_of_token,
                           pos_of_token, block_table, (float *)k_cache, (float *)v_cache, tab, sh);
    else
        hipLaunchKernelGGL(rope_kv_kernel<bf16_t>, grid, dim3(256), 0, s, (bf16_t *)qkv, seq_of_token,
                           pos_of_token, block_table, (bf16_t *)k_cache, (bf16_t *)v_cache, tab, sh);
    return hipGetLastError();
}

// ------------------------------------------------------------------ SiLU gate
// out[t, i] = g / (1 + exp(-g)) * u with g = gu[t, i], u = gu[t, I + i].
template <typename T>
__global__ __launch_bounds__(256) void silu_mul_kernel(const T *__restrict__ gu, T *__restrict__ out, int ld_out,
                                                       int I, size_t n_vec) {
    constexpr int V = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(V)));
    const int vec_per_row = I / V;
    for (size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x; idx < n_vec; idx += (size_t)gridDim.x * 256) {
        const size_t t = idx / vec_per_row, c = idx % vec_per_row;
        const vec_t g = *reinterpret_cast<const vec_t *>(gu + t * 2 * I + c * V);
        const vec_t u = *reinterpret_cast<const vec_t *>(gu + t * 2 * I + I + c * V);
        vec_t o;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float z = to_f32<T>(g[e]);
            o[e] = from_f32<T>(z / (1.0f + expf(-z)) * to_f32<T>(u[e]));
        }
        *reinterpret_cast<vec_t *>(out + t * ld_out + c * V) = o;
    }
}

// Split-K reduce of a gate/up projection fused with the gate (bf16): the planes of eight gate and of the eight up columns
// are summed in plane order and rounded - the values gemm_reduce_kernel would have stored - and gated as above.
// Bound by the planes' bytes, read once (two planes of 340 rows x 16384: 9.3 + 6.1 us as two launches, 9.9 us in one).
template <int SC>
__global__ __launch_bounds__(256) void gemm_reduce_gate_kernel(const float *__restrict__ P, size_t plane_stride, int S, bf16_t *__restrict__ out,
                                                               int ld_out, int I, size_t n_vec) {
    typedef bf16_t vec_t __attribute__((ext_vector_type(8)));
    const int vec_per_row = I / 8;
    for (size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x; idx < n_vec; idx += (size_t)gridDim.x * 256) {
        const size_t t = idx / vec_per_row, c = idx % vec_per_row;
        const float *p = P + t * 2 * I + c * 8;
        f32x4 v[4];                                        // gate, gate, up, up
        if constexpr (SC > 0) {                            // all plane loads in flight before the first add
            f32x4 l[SC][4];
#pragma unroll
            for (int sp = 0; sp < SC; ++sp)
#pragma unroll
                for (int j = 0; j < 4; ++j) l[sp][j] = *reinterpret_cast<const f32x4 *>(p + (size_t)sp * plane_stride + (j >> 1) * I + (j & 1) * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = l[0][j];
#pragma unroll
                for (int sp = 1; sp < SC; ++sp) { v[j][0] += l[sp][j][0]; v[j][1] += l[sp][j][1]; v[j][2] += l[sp][j][2]; v[j][3] += l[sp][j][3]; }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float *q = p + (j >> 1) * I + (j & 1) * 4;
                v[j] = *reinterpret_cast<const f32x4 *>(q);
                for (int sp = 1; sp < S; ++sp) {
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(q + (size_t)sp * plane_stride);
                    v[j][0] += a[0]; v[j][1] += a[1]; v[j][2] += a[2]; v[j][3] += a[3];
                }
            }
        }
        vec_t o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float z = bf2f(f2bf(v[e >> 2][e & 3])), u = bf2f(f2bf(v[2 + (e >> 2)][e & 3]));
            o[e] = f2bf(z / (1.0f + expf(-z)) * u);
        }
        *reinterpret_cast<vec_t *>(out + t * ld_out + c * 8) = o;
    }
}

bool reduce_gate_supported(int dtype, int I) { return dtype == 1 && I % 8 == 0; }

hipError_t launch_reduce_gate(const float *P, size_t plane_stride, int S, void *out, int ld_out, int rows, int I, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const size_t n_vec = (size_t)rows * (I / 8);
    const int blocks = (int)((n_vec + 255) / 256 < 4096 ? (n_vec + 255) / 256 : 4096);
#define DYN_RG(SC) hipLaunchKernelGGL(gemm_reduce_gate_kernel<SC>, dim3(blocks), dim3(256), 0, s, P, plane_stride, S, (bf16_t *)out, ld_out, I, n_vec)
    switch (S) {
        case 2: DYN_RG(2); break;
        case 4: DYN_RG(4); break;
        default: DYN_RG(0); break;
    }
#undef DYN_RG
    return hipGetLastError();
}

hipError_t launch_silu_mul(int dtype, const void *gu, void *out, int ld_out, int rows, int I, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int V = dtype == 0 ? 4 : 8;
    const size_t n_vec = (size_t)rows * (I / V);
    const int blocks = (int)((n_vec + 255) / 256 < 4096 ? (n_vec + 255) / 256 : 4096);
    if (dtype == 0)
        hipLaunchKernelGGL(silu_mul_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float *)gu, (float *)out, ld_out,
                           I, n_vec);
    else
        hipLaunchKernelGGL(silu_mul_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t *)gu,
                           (bf16_t *)out, ld_out, I, n_vec);
    return hipGetLastError();
}

// Read-only streaming probe: every 16-byte word of a buffer is loaded once (a workgroup reads
// 4 KB contiguously per step of a grid-wide stride; eight workgroups per CU keep the loads of
// different steps in flight) and folded into one word per wave so that the loads cannot be
// dropped.  What it reaches is the rate this GPU's memory system delivers to a kernel that does
// nothing else: the practical ceiling next to the datasheet peak.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4 *__restrict__ p, size_t n_vec, uint32_t *__restrict__ sink) {
    const size_t stride = (size_t)gridDim.x * 256;
    u32x4 acc = u32x4{0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += stride) acc ^= p[i];
    uint32_t v = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v ^= __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sink[blockIdx.x * 4 + (threadIdx.x >> 6)] = v;
}

constexpr int kProbeBlocks = 2048;      // eight workgroups for each of the 256 CUs

hipError_t launch_stream_read(const void *buf, size_t bytes, uint32_t *sink, hipStream_t s) {
    hipLaunchKernelGGL(stream_read_kernel, dim3(kProbeBlocks), dim3(256), 0, s, (const u32x4 *)buf, bytes / 16, sink);
    return hipGetLastError();
}

}  // namespace dyn
