// fp32 projections on fp32 MFMAs (launch_gemm and launch_gemm_grouped call launch_gemm_f32).
//
// K is cut into eight chains (kF32Chains slices of whole 16-deep units); each is accumulated by 16x16x4 fp32 MFMAs from
// zero, and the eight sums are added one after the other, then the residual: an output's order of terms follows
// from its column, N and K (and whether experts share the launch) alone, so its bits do not depend on the tile or on how
// many rows are in flight.
// Where K is a multiple of 512 and N of 4 a chain is whole blocks of 64 k (256 bytes of a row).  Product (r, e) of a block,
// r and e = 0..3, takes k = 16 c + 4 r + e as its k index c; the blocks of a chain are walked from one that turns with the
// chain and with the group of 64 columns, and the first chain added turns with that group too: rows lie a power of two
// apart, and what runs at the same time would otherwise read one channel of the second-level cache.
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"
#include "rotary.h"

namespace dyn {

constexpr int kF32Chains = 8, kF32Block = 64;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));       // weights, residual, output: any float alignment

__device__ __forceinline__ int f32_block(int i, int chain, int n0, int blocks) {     // the i-th block of a chain
    const int at = i + (chain + n0 / 64 * 3) % blocks;
    return at < blocks ? at : at - blocks;
}
__device__ __forceinline__ int f32_chain(int i, int n0) { return (i + n0 / 64) % kF32Chains; }     // the i-th chain to add

// Four outputs of a row from column n on: + residual, stored.
__device__ __forceinline__ void f32_store(f32x4 o, size_t at, int n, int N, const float *__restrict__ R, float *__restrict__ Y) {
    if (n + 4 <= N) {
        if (R) { const f32x4_u rv = *reinterpret_cast<const f32x4_u *>(R + at); o[0] += rv[0]; o[1] += rv[1]; o[2] += rv[2]; o[3] += rv[3]; }
        *reinterpret_cast<f32x4_u *>(Y + at) = o;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (n + r < N) Y[at + r] = o[r] + (R ? R[at + r] : 0.f);
    }
}

// What a tile of 32 W rows does when its first 16 (a = 0) and its other 16 (a = 1) are partners: nothing, gate columns and the up
// columns beside them, or head-dim indices and the ones half a head dim on, rotated and appended to the cache as
// rope_kv_vec_kernel does it.
struct F32Plain { static constexpr bool PAIRS = false, ROTARY = false; };
struct F32Gated { static constexpr bool PAIRS = true, ROTARY = false; int ldy; };
struct F32Rotary {
    static constexpr bool PAIRS = true, ROTARY = true;
    const int32_t *seq_of_token, *pos_of_token, *block_table;
    float *k_cache, *v_cache;
    RopeTable tab;
    AttnShape sh;
};
// First W row of a tile, and how far on its partners lie.
template <class EP>
__device__ __forceinline__ int f32_column(const EP &ep, int nt, int N, int &partner) {
    if constexpr (EP::ROTARY) {
        const int d = ep.sh.head_dim, per_head = d / 32;
        partner = d / 2;
        return (int)blockIdx.x / per_head * d + (int)blockIdx.x % per_head * 16;
    }
    partner = N / 2;
    return blockIdx.x * (EP::PAIRS ? nt / 2 : nt);
}
// Rotary: a wave takes one angle a lane, angle r of the 16 rows b = wave % NB, before its operands are multiplied, and looks the page up.
template <int NB>
struct F32Angles { float2 at[NB][4][64]; };
template <int NB>
__device__ __forceinline__ void f32_angles(F32Angles<NB> &angles, const F32Rotary &ep, int m0, int n0, int M, int &pos, int &page) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b = wave % NB, r = wave / NB;
    const int m = min(m0 + b * 16 + (lane & 15), M - 1);
    pos = ep.pos_of_token[m];
    page = ep.block_table[(size_t)ep.seq_of_token[m] * ep.sh.max_pages_per_seq + pos / ep.sh.page_size];
    if (r >= 4) return;
    float s, c;
    rotary_angle(pos, ep.tab.inv_freq[n0 % ep.sh.head_dim + 4 * (lane >> 4) + r], s, c);
    angles.at[b][r][lane] = make_float2(c, s);
}

// NORM: X rows are normalised as they are loaded, x * r * g with rmsnorm_row's r, where the launch has one workgroup row or few: a norm's
// own launch is as long as reading one row twice, and every workgroup reads the rows anyway.
struct F32Norm { const float *g; float eps; };

// The rows' sums of squares as rmsnorm_row takes them, a row to each half of the workgroup, P of them at a time; then r of row `row` of the tile.
template <int P>
__device__ __forceinline__ void f32_squares(float (*part)[4], const float *__restrict__ X, int ldx, int m0, int M, int K) {
    const int half = threadIdx.x >> 8, tid = threadIdx.x & 255;
    float ss[P];
#pragma unroll
    for (int p = 0; p < P; ++p) ss[p] = 0.f;
    for (int i = tid; i < K / 4; i += 256) {
        f32x4 v[P];
#pragma unroll
        for (int p = 0; p < P; ++p) v[p] = *reinterpret_cast<const f32x4_u *>(X + (size_t)min(m0 + 2 * p + half, M - 1) * ldx + 4 * i);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) ss[p] = __builtin_fmaf(v[p][e], v[p][e], ss[p]);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        ss[p] = wave_sum(ss[p]);
        if ((tid & 63) == 0) part[2 * p + half][tid >> 6] = ss[p];
    }
}
__device__ __forceinline__ void f32_row_squares(float (*part)[4], const float *__restrict__ X, int ldx, int m0, int M, int K) {
    const int rows = M - m0;
    if (rows <= 4) f32_squares<2>(part, X, ldx, m0, M, K);
    else if (rows <= 8) f32_squares<4>(part, X, ldx, m0, M, K);
    else f32_squares<8>(part, X, ldx, m0, M, K);
    __syncthreads();
}
__device__ __forceinline__ float f32_row_scale(const float (*part)[4], int row, int K, float eps) {
    const float total = ((part[row][0] + part[row][1]) + part[row][2]) + part[row][3];
    return 1.0f / sqrtf(total / (float)K + eps);
}

// silu(g) * u
__device__ __forceinline__ f32x4 f32_gate(f32x4 g, f32x4 u) {
    f32x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = g[r] / (1.0f + expf(-g[r])) * u[r];
    return o;
}

// The eight waves' sums of a tile meet in LDS, SUB sub-tiles of 16 x 16 at a time, a wave to a sub-tile or to a pair of partners.
// D: lane l holds W rows 4 (l / 16) + r of X row l % 16.  list: output rows (null: m itself).
template <int NA, int NB, bool TURN, class EP>
__device__ __forceinline__ void f32_finish(f32x4 (*part)[NA * NB < 4 ? NA * NB : 4][64], const f32x4 (&acc)[NA][NB], int m0, int n0, int M, int N,
                                           const int32_t *list, const float *__restrict__ R, float *__restrict__ Y, const EP &ep,
                                           const F32Angles<NB> *angles, int pos, int page) {
    constexpr int SUB = NA * NB < 4 ? NA * NB : 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
    if constexpr (EP::PAIRS) {
        static_assert(NA == 2 && SUB == NA * NB, "one pair of sub-tiles per 16 rows of X");
#pragma unroll
        for (int i = 0; i < SUB; ++i) part[wave][i][lane] = acc[i / NB][i % NB];
        __syncthreads();
        if (wave >= NB) return;
        f32x4 g = part[TURN ? f32_chain(0, n0) : 0][wave][lane], u = part[TURN ? f32_chain(0, n0) : 0][NB + wave][lane];
#pragma unroll
        for (int w = 1; w < kF32Chains; ++w) {
            const f32x4 p = part[TURN ? f32_chain(w, n0) : w][wave][lane], q = part[TURN ? f32_chain(w, n0) : w][NB + wave][lane];
            g[0] += p[0]; g[1] += p[1]; g[2] += p[2]; g[3] += p[3];
            u[0] += q[0]; u[1] += q[1]; u[2] += q[2]; u[3] += q[3];
        }
        const int m = m0 + wave * 16 + lr;
        if (m >= M) return;
        if constexpr (EP::ROTARY) {
            const AttnShape &sh = ep.sh;
            const int d = sh.head_dim, head = n0 / d, i = n0 % d + 4 * lq, slot = pos % sh.page_size;
            if (head >= sh.n_q + sh.n_kv) {                // v head -> V page [kvh][d][slot]
                float *vp = ep.v_cache + (((size_t)page * sh.n_kv + (head - sh.n_q - sh.n_kv)) * d + i) * sh.page_size + slot;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    vp[(size_t)r * sh.page_size] = g[r];
                    vp[(size_t)(r + d / 2) * sh.page_size] = u[r];
                }
                return;
            }
            f32x4 lo, hi;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 cs = angles->at[wave][r][lane];
                lo[r] = rotated_lo(g[r], u[r], cs.x, cs.y);
                hi[r] = rotated_hi(g[r], u[r], cs.x, cs.y);
            }
            float *dst = head < sh.n_q ? Y + (size_t)m * N + head * d : ep.k_cache + (((size_t)page * sh.n_kv + (head - sh.n_q)) * sh.page_size + slot) * d;
            *reinterpret_cast<f32x4_u *>(dst + i) = lo;
            *reinterpret_cast<f32x4_u *>(dst + i + d / 2) = hi;
        } else {
            *reinterpret_cast<f32x4_u *>(Y + (size_t)m * ep.ldy + n0 + 4 * lq) = f32_gate(g, u);
        }
        return;
    }
#pragma unroll
    for (int s0 = 0; s0 < NA * NB; s0 += SUB) {
        if (s0) __syncthreads();
#pragma unroll
        for (int i = 0; i < SUB; ++i) part[wave][i][lane] = acc[(s0 + i) / NB][(s0 + i) % NB];
        __syncthreads();
        if (wave < SUB) {
            const int a = (s0 + wave) / NB, b = (s0 + wave) % NB;
            f32x4 o = part[TURN ? f32_chain(0, n0) : 0][wave][lane];
#pragma unroll
            for (int w = 1; w < kF32Chains; ++w) { const f32x4 p = part[TURN ? f32_chain(w, n0) : w][wave][lane]; o[0] += p[0]; o[1] += p[1]; o[2] += p[2]; o[3] += p[3]; }
            const int m = m0 + b * 16 + lr, n = n0 + a * 16 + 4 * lq;
            if (m < M && n < N) f32_store(o, (size_t)(list ? list[m] : m) * N + n, n, N, R, Y);
        }
    }
}

// Any shape: eight waves share one MT (X rows) x NT (W rows) output tile, a wave per chain.
// Operands go from memory straight into MFMA layout: a lane loads four consecutive k of its row (16
// rows x 64 bytes per instruction) and element e of the four is the operand of product e, whose k
// index l / 16 then stands for k 4 (l / 16) + e in both matrices.  Launch alone, against 64 x 64 tiles of fp32 FMAs staged
// through LDS 16 k at a time by one chain per output: 4 rows x 768 x 256 27.7 -> 3.2 us, 4 x 256 x 1024 96 -> 5.1 us.
template <int MT, int NT, bool NORM, class EP>
__global__ __launch_bounds__(kF32Chains * 64) void gemm_f32_kernel(const float *__restrict__ X, int ldx, const float *__restrict__ W,
                                                                  const float *__restrict__ R, float *__restrict__ Y, int M, int N,
                                                                  int K, GemmGroups gr, F32Norm norm, EP ep) {
    static_assert(!NORM || MT == 16, "a lane has one X row");
    __shared__ float squares[NORM ? 16 : 1][4];
    constexpr int NA = NT / 16, NB = MT / 16, UNR = (NA + NB) <= 4 ? 4 : 2;  // units of 16 k loaded ahead of their products
    __shared__ f32x4 part[kF32Chains][NA * NB < 4 ? NA * NB : 4][64];
    __shared__ F32Angles<EP::ROTARY ? NB : 1> angles;
    const int32_t *list = nullptr;
    if (gr.n_groups) {                                 // blockIdx.z = expert: its rows come from a list
        M = gr.counts[blockIdx.z];
        list = gr.lists + (size_t)blockIdx.z * gr.cap;
        W += (size_t)blockIdx.z * gr.w_stride;
    }
    const int m0 = blockIdx.y * MT;
    if (m0 >= M) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
    int partner, pos = 0, page = 0;
    const int n0 = f32_column(ep, NT, N, partner);
    const float *wp[NA], *xp[NB];                      // rows past the end read the last one; what they give is not stored
#pragma unroll
    for (int a = 0; a < NA; ++a) wp[a] = W + (size_t)(EP::PAIRS ? n0 + a * partner + lr : min(n0 + a * 16 + lr, N - 1)) * K + 4 * lq;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int m = min(m0 + b * 16 + lr, M - 1);
        xp[b] = X + (size_t)(list ? list[m] / gr.x_div : m) * ldx + 4 * lq;
    }
    f32x4 acc[NA][NB];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int units = (K + 15) / 16, u0 = units * wave / kF32Chains, u1 = units * (wave + 1) / kF32Chains;
    const int full = K / 16;                           // whole units; the last one of a K that is no multiple of 16 is read guarded
    auto multiply = [&](const f32x4 (&wv)[NA], const f32x4 (&xv)[NB]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[a][e], xv[b][e], acc[a][b], 0, 0, 0);
    };
    int u = u0;
    const int u1f = min(u1, full);
    if constexpr (NORM) {                              // K is a multiple of 256: a chain has an even number of units, two at a time here
        f32x4 wv[2][NA], xv[2][NB], gv[2];
        auto load = [&](int at) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int a = 0; a < NA; ++a) wv[i][a] = *reinterpret_cast<const f32x4_u *>(wp[a] + (size_t)(at + i) * 16);
                xv[i][0] = *reinterpret_cast<const f32x4_u *>(xp[0] + (size_t)(at + i) * 16);
                gv[i] = *reinterpret_cast<const f32x4_u *>(norm.g + (at + i) * 16 + 4 * lq);
            }
        };
        load(u);                                       // on its way while the sums of squares are taken
        if constexpr (EP::ROTARY) f32_angles(angles, ep, m0, n0, M, pos, page);
        f32_row_squares(squares, X, ldx, m0, M, K);
        const float r = f32_row_scale(squares, min(lr, M - 1 - m0), K, norm.eps);
        while (true) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) xv[i][0][e] = xv[i][0][e] * r * gv[i][e];
                multiply(wv[i], xv[i]);
            }
            u += 2;
            if (u >= u1) break;
            load(u);
        }
    } else if constexpr (EP::ROTARY) {
        f32_angles(angles, ep, m0, n0, M, pos, page);
    }
    auto batch = [&](auto n) {                         // n units, their loads together
        constexpr int U = decltype(n)::value;
        f32x4 wv[U][NA], xv[U][NB];
#pragma unroll
        for (int i = 0; i < U; ++i) {
#pragma unroll
            for (int a = 0; a < NA; ++a) wv[i][a] = *reinterpret_cast<const f32x4_u *>(wp[a] + (size_t)(u + i) * 16);
#pragma unroll
            for (int b = 0; b < NB; ++b) xv[i][b] = *reinterpret_cast<const f32x4_u *>(xp[b] + (size_t)(u + i) * 16);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) multiply(wv[i], xv[i]);
        u += U;
    };
    while (u + UNR <= u1f) batch(std::integral_constant<int, UNR>());
    if (UNR > 2 && u + 2 <= u1f) batch(std::integral_constant<int, 2>());
    for (; u < u1; ++u) {
        f32x4 wv[NA], xv[NB];
        const bool in = u < full || u * 16 + 4 * lq < K;            // K is a multiple of 4
#pragma unroll
        for (int a = 0; a < NA; ++a) wv[a] = in ? (f32x4) * reinterpret_cast<const f32x4_u *>(wp[a] + (size_t)u * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < NB; ++b) xv[b] = in ? (f32x4) * reinterpret_cast<const f32x4_u *>(xp[b] + (size_t)u * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
        multiply(wv, xv);
    }
    f32_finish<NA, NB, false>(part, acc, m0, n0, M, N, list, R, Y, ep, EP::ROTARY ? (const F32Angles<NB> *)&angles : nullptr, pos, page);
}

// Four adjacent lanes trade with four registers: register j of lane x of every quad becomes register x of lane j.
__device__ __forceinline__ void quad_transpose(f32x4 (&v)[4]) {
    const bool x0 = threadIdx.x & 1, x1 = threadIdx.x & 2;
#define DYN_TRADE(A, B, CTRL, UP)                                                                         \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                       \
        const int a = __float_as_int(v[A][e]), b = __float_as_int(v[B][e]);                               \
        const int an = __builtin_amdgcn_mov_dpp(a, CTRL, 0xf, 0xf, true), bn = __builtin_amdgcn_mov_dpp(b, CTRL, 0xf, 0xf, true); \
        v[A][e] = __int_as_float(UP ? bn : a);                                                            \
        v[B][e] = __int_as_float(UP ? b : an);                                                            \
    }
    DYN_TRADE(0, 1, 0xb1, x0)                              // quad_perm 1, 0, 3, 2
    DYN_TRADE(2, 3, 0xb1, x0)
    DYN_TRADE(0, 2, 0x4e, x1)                              // quad_perm 2, 3, 0, 1
    DYN_TRADE(1, 3, 0x4e, x1)
#undef DYN_TRADE
}

// Whole blocks, few rows or few tiles: as above, but a quad of lanes loads 64 adjacent bytes and trades them.  Load j of a
// block's four covers rows 4 q + j, q = 0..3, 256 bytes each; in MFMA layout a quarter wave names 16 rows and the
// load takes 65 cycles of the vector cache, this way 17.  16 x 16 tiles keep two blocks in flight (24 rows x 1024 x 4096
// 15.9 -> 11.0 us, 100 rows 30.7 -> 19.2); with 32 x 32 that costs the second workgroup of a CU (225 rows x 1024 x 4096 31.6 -> 28.8
// us, 30.3 with two).  Trading takes 64 vector instructions an operand.  Up to 8 rows X is loaded straight into MFMA layout instead (XQUADS
// false): the lanes of rows past the last one name its lines again, so a load costs what its few rows do (1 / 4 rows: 8192 x 1024, gated 11.9 /
// 12.7 -> 11.9 / 11.9 us, 1024 x 4096 11.2 / 11.0 -> 9.7 / 9.8, 16384 x 2048, gated 28.2 / 28.4 -> 23.4 / 24.2, 2048 x 8192 20.2 / 20.4 ->
// 17.1 / 18.3; steps of 2048 wide, 8192 MLP, 1 / 8 / 16 rows 92.7 / 98.2 / 99.2 -> 84.5 / 92.1 / 99.0: at 16 rows either way, so the line is
// where half the rows are there).
template <int MT, int NT, bool XQUADS, bool NORM, class EP>
__global__ __launch_bounds__(kF32Chains * 64) void gemm_f32_quads_kernel(const float *__restrict__ X, int ldx, const float *__restrict__ W,
                                                                        const float *__restrict__ R, float *__restrict__ Y, int M, int N, int K,
                                                                        F32Norm norm, EP ep) {
    static_assert(!NORM || MT == 16, "a tile of few rows");
    __shared__ float squares[NORM ? 16 : 1][4];
    constexpr int NA = NT / 16, NB = MT / 16, NBUF = NA + NB <= 3 ? 2 : 1;
    __shared__ f32x4 part[kF32Chains][NA * NB < 4 ? NA * NB : 4][64];
    __shared__ F32Angles<EP::ROTARY ? NB : 1> angles;
    int partner, pos = 0, page = 0;
    const int m0 = blockIdx.y * MT, n0 = f32_column(ep, NT, N, partner);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), row4 = (lane >> 2 & 3) * 4, col = (lane >> 4) * 16 + (lane & 3) * 4;
    const float *const Wt = W + (size_t)n0 * K, *const Xt = X + (size_t)m0 * ldx;
    size_t wo[NA], xo[NB][4];                              // rows past the end read the last ones; what they give is not stored
#pragma unroll
    for (int a = 0; a < NA; ++a) wo[a] = (size_t)(EP::PAIRS ? a * partner + row4 : min(a * 16 + row4, N - 4 - n0)) * K + col;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) xo[b][j] = XQUADS ? (size_t)min(b * 16 + row4 + j, M - 1 - m0) * ldx + col : (size_t)min(b * 16 + (lane & 15), M - 1 - m0) * ldx + (lane >> 4) * 16 + 4 * j;
    f32x4 acc[NA][NB];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int blocks = K / (kF32Block * kF32Chains);
    f32x4 wv[NBUF][NA][4], xv[NBUF][NB][4], gv[NORM ? NBUF : 1][XQUADS ? 1 : 4];
    float scale[XQUADS ? 4 : 1];                           // of the rows of this lane's X loads
    auto load = [&](auto buf, int i) {
        constexpr int B = decltype(buf)::value;
        const int at = (wave * blocks + f32_block(i, wave, n0, blocks)) * kF32Block;
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int j = 0; j < 4; ++j) wv[B][a][j] = *reinterpret_cast<const f32x4_u *>(Wt + (size_t)j * K + at + wo[a]);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[B][b][j] = *reinterpret_cast<const f32x4_u *>(Xt + at + xo[b][j]);
        if constexpr (NORM) {
#pragma unroll
            for (int j = 0; j < (XQUADS ? 1 : 4); ++j) gv[B][j] = *reinterpret_cast<const f32x4_u *>(norm.g + at + (XQUADS ? col : (lane >> 4) * 16 + 4 * j));
        }
    };
    auto multiply = [&](auto buf) {
        constexpr int B = decltype(buf)::value;
        if constexpr (NORM) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) xv[B][0][j][e] = xv[B][0][j][e] * scale[XQUADS ? j : 0] * gv[B][XQUADS ? 0 : j][e];
        }
#pragma unroll
        for (int a = 0; a < NA; ++a) quad_transpose(wv[B][a]);
        if constexpr (XQUADS) {
#pragma unroll
            for (int b = 0; b < NB; ++b) quad_transpose(xv[B][b]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[B][a][r][e], xv[B][b][r][e], acc[a][b], 0, 0, 0);
    };
    const std::integral_constant<int, 0> b0;
    const std::integral_constant<int, NBUF - 1> b1;
    if constexpr (NBUF == 1) {
        if constexpr (EP::ROTARY) f32_angles(angles, ep, m0, n0, M, pos, page);
        for (int i = 0; i < blocks; ++i) {
            load(b0, i);
            multiply(b0);
        }
    } else {                                               // a pass always loads: behind a load that may not have been issued the compiler waits for all
        load(b0, 0);
        if constexpr (EP::ROTARY) f32_angles(angles, ep, m0, n0, M, pos, page);
        if constexpr (NORM) {                              // while the first block is on its way
            f32_row_squares(squares, X, ldx, m0, M, K);
#pragma unroll
            for (int j = 0; j < (XQUADS ? 4 : 1); ++j) scale[j] = f32_row_scale(squares, min(XQUADS ? row4 + j : (lane & 15), M - 1 - m0), K, norm.eps);
        }
        int i = 0;
        for (; i + 2 < blocks; i += 2) {
            load(b1, i + 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(b0);
            __builtin_amdgcn_sched_barrier(0);
            load(b0, i + 2);
            __builtin_amdgcn_sched_barrier(0);
            multiply(b1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (i + 1 < blocks) {
            load(b1, i + 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(b0);
            multiply(b1);
        } else {
            multiply(b0);
        }
    }
    f32_finish<NA, NB, true>(part, acc, m0, n0, M, N, nullptr, R, Y, ep, EP::ROTARY ? (const F32Angles<NB> *)&angles : nullptr, pos, page);
}

// Whole blocks, many tiles: 64 x 64, four waves of 32 x 32 that share stages of one block (256-byte rows, direct loads of
// one row per quarter wave, two stages) and walk the chains one after the other, each chain's sum added to the
// total in registers.  Two workgroups per CU, bound by the matrix rate and the first stage's latency: 100 / 225 / 300 rows x 8192 x
// 1024 31 / 56.5 / 79 us with 64 x 64 tiles loaded straight into MFMA layout (eight waves, 16 rows a quarter wave) -> 24.5 /
// 41.2 / 60.5.  The 16-byte columns are swizzled with the row: lanes of 16 rows read 16
// different bank groups.
// GATED: of every 32 W rows of the tile the first 16 are gate columns and the other 16 the up columns beside them.
constexpr int kF32TileLds = 2 * 128 * 256;
template <bool GATED>
__global__ __launch_bounds__(256, 2) void gemm_f32_tiles_kernel(const float *__restrict__ X, int ldx, const float *__restrict__ W,
                                                                const float *__restrict__ R, float *__restrict__ Y, int M, int N, int K, int ldy) {
    constexpr int T = 64, LOADS = 2 * T / 4 / 4, STAGE = 2 * T * 256;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int m0 = blockIdx.y * T, n0 = blockIdx.x * (GATED ? T / 2 : T);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
    const int wn = wave & 1, wm = wave >> 1;
    const int blocks = K / (kF32Block * kF32Chains), n_stage = kF32Chains * blocks;
    const float *src[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int row = (j * 4 + wave) * 4 + (lane >> 4), col = ((lane ^ row) & 15) * 4;
        const int n = GATED ? n0 + (row >> 5) * 16 + (row & 15) + (row & 16 ? N / 2 : 0) : min(n0 + row, N - 1);
        src[j] = row < T ? W + (size_t)n * K + col : X + (size_t)min(m0 + row - T, M - 1) * ldx + col;
    }
    int at_chain = 0, at_block = 0;                        // next stage to issue
    auto issue = [&](int st) {
        const int chain = f32_chain(at_chain, n0), k = (chain * blocks + f32_block(at_block, chain, n0, blocks)) * kF32Block;
        if (++at_block == blocks) { at_block = 0; ++at_chain; }
#pragma unroll
        for (int j = 0; j < LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + k),
                                             (__attribute__((address_space(3))) void *)(lds + (st & 1) * STAGE + (j * 4 + wave) * 1024), 16, 0, 0);
    };
    f32x4 acc[2][2], total[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    issue(0);
    int left = blocks;                                     // stages left of the chain
    bool first = true;
    for (int st = 0; st < n_stage; ++st) {
        wait_vmcnt(0);
        // Bare barrier: every wave sees stage st and has its operands of the one before in registers.
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (st + 1 < n_stage) issue(st + 1);
        const unsigned char *buf = lds + (st & 1) * STAGE;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 wv[2], xv[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) { const int row = wn * 32 + a * 16 + lr; wv[a] = *reinterpret_cast<const f32x4 *>(buf + row * 256 + (((lq * 4 + r) ^ lr) << 4)); }
#pragma unroll
            for (int b = 0; b < 2; ++b) { const int row = T + wm * 32 + b * 16 + lr; xv[b] = *reinterpret_cast<const f32x4 *>(buf + row * 256 + (((lq * 4 + r) ^ lr) << 4)); }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[a][e], xv[b][e], acc[a][b], 0, 0, 0);
        }
        if (--left == 0) {                                 // the chain ends
            left = blocks;
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (first) total[a][b] = acc[a][b];
                    else { total[a][b][0] += acc[a][b][0]; total[a][b][1] += acc[a][b][1]; total[a][b][2] += acc[a][b][2]; total[a][b][3] += acc[a][b][3]; }
                    acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            first = false;
        }
    }
    if constexpr (GATED) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int m = m0 + wm * 32 + b * 16 + lr;
            if (m < M) *reinterpret_cast<f32x4_u *>(Y + (size_t)m * ldy + n0 + wn * 16 + 4 * lq) = f32_gate(total[0][b], total[1][b]);
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int m = m0 + wm * 32 + b * 16 + lr, n = n0 + wn * 32 + a * 16 + 4 * lq;
            if (m < M && n < N) f32_store(total[a][b], (size_t)m * N + n, n, N, R, Y);
        }
}

// Tile of an fp32 launch.  16 x 16 up to 16 rows or 512 tiles, two a CU: the launch is as long as a workgroup, and a workgroup's
// products take a time of their own (whole blocks, 32 x 32 -> 16 x 16: 48 rows x 1536 x 1024, 288 tiles, 8.7 -> 7.0 us; 100 x 1024 x 4096,
// 448 tiles, 27.9 -> 19.2; past the line 160 x 1024 x 4096, 640 tiles, 28.4 -> 28.7, 24 x 8192 x 1024, 1024 tiles, 13.2 -> 15.5).  64 x 64
// where such tiles are about a CU's each: 192 of them (225 rows x 8192 x 1024, 512 tiles: 41 us; 225 x 1536 x 1024, 96 tiles: 23.5 us, with
// 32 x 32 17.1).  Else 32 x 32.  Other depths and widths, and experts, take the form for any shape.
//
// The gated form takes the same tiles over all 2 I columns; its 16-row tile is 16 gate and 16 up columns wide.  It exists for any number of rows for whole
// blocks and I a multiple of 32; the launch it saves and the [gate | up] rows' way through memory are 5.8 us of a step of 225 rows (1024
// wide, 4096 MLP: 136.9 -> 131.1 us).
namespace {
template <bool GATED>
hipError_t launch_f32_tiles(const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int ldy, hipStream_t s) {
    static bool attr_set = false;                      // 64 KB of dynamic LDS: opted in, once
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)gemm_f32_tiles_kernel<GATED>, hipFuncAttributeMaxDynamicSharedMemorySize, kF32TileLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(gemm_f32_tiles_kernel<GATED>, dim3((N + 63) / 64, (rows + 63) / 64), dim3(256), kF32TileLds, s, (const float *)X, ldx,
                       (const float *)W, (const float *)R, (float *)Y, rows, N, K, ldy);
    return hipGetLastError();
}

template <int MT, int NT, class EP>
hipError_t launch_f32_quads(const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, const F32Norm &norm, const EP &ep,
                            hipStream_t s) {
#define DYN_QUADS(XQUADS, NORM)                                                                                                                 \
    hipLaunchKernelGGL((gemm_f32_quads_kernel<MT, NT, XQUADS, NORM, EP>), dim3((N + NT - 1) / NT, (rows + MT - 1) / MT), dim3(kF32Chains * 64), 0, s, \
                       (const float *)X, ldx, (const float *)W, (const float *)R, (float *)Y, rows, N, K, norm, ep)
    if constexpr (MT == 16) {
        if constexpr (EP::PAIRS)
            if (norm.g) {
                if (rows <= 8) DYN_QUADS(false, true);
                else DYN_QUADS(true, true);
                return hipGetLastError();
            }
        if (rows <= 8) {
            DYN_QUADS(false, false);
            return hipGetLastError();
        }
    }
    DYN_QUADS(true, false);
#undef DYN_QUADS
    return hipGetLastError();
}

long f32_tiles(int rows, int N, int t) { return (long)((rows + t - 1) / t) * ((N + t - 1) / t); }
bool f32_whole(int N, int K) { return K % (kF32Block * kF32Chains) == 0 && N % 4 == 0; }
bool f32_few(int rows, int N, bool whole, int groups = 1) { return rows <= 16 || f32_tiles(rows, N, 16) * groups <= (whole ? 512 : 256); }
bool f32_direct(const void *X, int ldx, const void *W, int rows, int N) {      // 64 x 64 tiles; the direct loads take 16 bytes
    return ldx % 4 == 0 && (((uintptr_t)X | (uintptr_t)W) & 15) == 0 && f32_tiles(rows, N, 64) >= 192;
}

int f32_pitch(const F32Plain &, int N) { return N; }
int f32_pitch(const F32Gated &ep, int) { return ep.ldy; }

template <class EP>
hipError_t launch_f32_whole(const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, const F32Norm &norm, const EP &ep,
                            hipStream_t s) {
    if (f32_few(rows, N, true)) return launch_f32_quads<16, EP::PAIRS ? 32 : 16>(X, ldx, W, R, Y, rows, N, K, norm, ep, s);
    if constexpr (!EP::ROTARY)
        if (f32_direct(X, ldx, W, rows, N)) return launch_f32_tiles<EP::PAIRS>(X, ldx, W, R, Y, rows, N, K, f32_pitch(ep, N), s);
    return launch_f32_quads<32, 32>(X, ldx, W, R, Y, rows, N, K, norm, ep, s);
}

template <int MT, int NT, class EP>
hipError_t launch_f32_any(const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, const GemmGroups &gr, const EP &ep,
                          hipStream_t s, const F32Norm &norm = F32Norm{nullptr, 0.f}) {
#define DYN_ANY(NORM)                                                                                                                                  \
    hipLaunchKernelGGL((gemm_f32_kernel<MT, NT, NORM, EP>), dim3((N + NT - 1) / NT, (rows + MT - 1) / MT, std::max(gr.n_groups, 1)), dim3(kF32Chains * 64), \
                       0, s, (const float *)X, ldx, (const float *)W, (const float *)R, (float *)Y, rows, N, K, gr, norm, ep)
    if constexpr (MT == 16 && EP::PAIRS)
        if (norm.g) {
            DYN_ANY(true);
            return hipGetLastError();
        }
    DYN_ANY(false);
#undef DYN_ANY
    return hipGetLastError();
}
}  // namespace

hipError_t launch_gemm_f32(const void *X, int ldx, const void *W, const void *R, void *Y, int max_rows, int N, int K,
                           const GemmGroups &gr, hipStream_t s) {
    if (!gr.n_groups && f32_whole(N, K)) return launch_f32_whole(X, ldx, W, R, Y, max_rows, N, K, F32Norm{nullptr, 0.f}, F32Plain{}, s);
    const int groups = std::max(gr.n_groups, 1);
    if (f32_few(max_rows, N, false, groups)) return launch_f32_any<16, 16>(X, ldx, W, R, Y, max_rows, N, K, gr, F32Plain{}, s);
    if (f32_tiles(max_rows, N, 64) * groups >= 256) return launch_f32_any<64, 64>(X, ldx, W, R, Y, max_rows, N, K, gr, F32Plain{}, s);
    return launch_f32_any<32, 32>(X, ldx, W, R, Y, max_rows, N, K, gr, F32Plain{}, s);
}

// (From I = 64 on: a narrower activation's padded rows are longer than [gate | up] rows, and a plan's workspace would grow.)
bool gemm_f32_gated_supported(int N2, int K) { return f32_whole(N2, K) && N2 % 64 == 0 && N2 >= 128; }

// Other depths: tiles of 16 + 16 columns, few rows or few tiles (a step of 256 wide, 4 / 32 rows 39.4 / 45.9 -> 37.8 / 43.7 us; 768 wide, 8 rows 60.2 -> 56.6).
bool gemm_f32_gated_rows_supported(int rows, int N2, int K) {
    return gemm_f32_gated_supported(N2, K) || (N2 % 64 == 0 && N2 >= 128 && !f32_whole(N2, K) && f32_few(rows, N2, false));
}

// The norm in the same launch: rows of up to 1024, 8192 elements of X in all, the step with norms of their own -> in the projections: 256 wide 1 / 8 /
// 16 / 32 rows 36.1 / 42.3 / 43.4 / 43.8 -> 32.7 / 38.8 / 41.4 / 41.8 us; 512 wide 1 / 8 / 16 rows 41.1 / 47.4 / 48.6 -> 37.8 / 44.7 / 47.8; 1024
// wide 1 / 4 / 8 rows 47.3 / 49.0 / 49.9 -> 45.3 / 46.8 / 49.3.  Beyond, a workgroup's own pass over X is longer than the launch: 512 wide 24
// rows 48.4 -> 48.6, 1024 wide 16 rows 52.2 -> 54.4, 2048 wide 1 / 8 rows 84.6 / 91.5 -> 87.3 / 97.3, 4096 wide 8 rows 163 -> 166.
// Every workgroup makes that pass, so it is one that each CU (n_cus of them, 0: 256) makes once, twice where a pass is short (any depth, up to 768 wide here).
// Steps, norms of their own -> inside: 1024 wide, 8192 MLP (512 tiles) 1 / 4 / 8 rows 55.5 / 57.6 / 63.4 -> 57.5 / 59.8 / 66.1, 16384 MLP 82.1 / 86.7 / 93.6 -> 85.8 /
// 91.0 / 100.5; 512 wide, 8192 MLP, 10 / 16 rows 57.6 / 58.5 -> 60.9 / 61.6; 1024 wide, 4096 MLP (256 tiles) on 64 CUs 1 / 8 rows 81.8 / 91.5 -> 89.3 / 101.4; but 256 and
// 768 wide, 8192 MLP (512 tiles) 46.0 -> 42.3 and 56.4 -> 52.1 at 4 rows.
bool gemm_f32_norm_supported(int rows, int N, int K, int n_cus) {
    const bool whole = f32_whole(N, K);
    const long tiles = (long)((rows + 15) / 16) * ((N + 31) / 32);
    return K % 256 == 0 && K <= 1024 && (long)rows * K <= 8192 && f32_few(rows, N, whole) && tiles <= (whole ? 1 : 2) * (n_cus > 0 ? n_cus : 256);
}

hipError_t launch_gemm_f32_gated(const void *X, int ldx, const void *W, void *Y, int ldy, int rows, int N2, int K, const GemmNorm &norm, hipStream_t s) {
    const F32Norm nm{(const float *)norm.g, norm.eps};
    if (f32_whole(N2, K)) return launch_f32_whole(X, ldx, W, nullptr, Y, rows, N2, K, nm, F32Gated{ldy}, s);
    return launch_f32_any<16, 32>(X, ldx, W, nullptr, Y, rows, N2, K, GemmGroups{}, F32Gated{ldy}, s, nm);
}

// The rotary form: tiles of 16 + 16 columns for few rows or few tiles at any depth, and 32 x 32 of whole blocks, where a
// head's halves have to lie in one group of 64 columns.  225 rows x 1536 x 1024 17.8 + 4.9 us as two launches, 19.3 in one; 4 rows x 768 x
// 256 3.3 + 2.7 -> 4.4 (steps 131.1 -> 128.5, 40.5 -> 39.2 us).
bool gemm_f32_rope_supported(const void *X, int ldx, const void *W, int rows, int N, int K, const AttnShape &sh) {
    if (sh.head_dim % 32 || sh.head_dim > 2 * kMaxHalfDim) return false;
    if (!f32_whole(N, K)) return f32_few(rows, N, false);
    return 64 % sh.head_dim == 0 && (f32_few(rows, N, true) || !f32_direct(X, ldx, W, rows, N));
}

hipError_t launch_gemm_f32_rope(const void *X, int ldx, const void *W, void *Y, int rows, int N, int K, const GemmNorm &norm, const GemmEpilogue &rope,
                                hipStream_t s) {
    const F32Norm nm{(const float *)norm.g, norm.eps};
    const F32Rotary ep{rope.seq_of_token, rope.pos_of_token, rope.block_table, (float *)rope.k_cache, (float *)rope.v_cache, *rope.rope, *rope.shape};
    if (f32_whole(N, K)) return launch_f32_whole(X, ldx, W, nullptr, Y, rows, N, K, nm, ep, s);
    return launch_f32_any<16, 32>(X, ldx, W, nullptr, Y, rows, N, K, GemmGroups{}, ep, s, nm);
}

}  // namespace dyn
