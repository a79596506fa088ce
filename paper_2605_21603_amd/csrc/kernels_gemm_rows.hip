// bf16 projections with planes for up to 16 rows: the planes summed inside the workgroup.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "gemm_tile.h"
#include "kernels.h"
#include "rotary.h"

namespace dyn {

// A workgroup owns 16 W rows over the whole depth, wave p plane p of the S, and the planes meet in LDS.  Bound by the weight
// stream; what it saves is the planes' way through memory and the launch that sums them.  The stages of a plane are walked in
// the rotated order of the other tiles and the planes are added in plane order: the same bits.
// W and X go into a ring of the wave's own by direct loads of whole 128-byte lines, and come out in MFMA layout: loaded straight
// into that layout a quarter wave names 16 rows, which costs 65 cycles of the vector cache an instruction against 17, and at 8
// rows X's loads and W's together took longer than W's way from memory.  No barrier in the loop, kDeep stages on their way
// (64 KB a CU with 8 planes; 5: no change).  Launch alone, straight -> by LDS, weights from HBM / from the last-level cache:
// 6144 x 4096 1 row 12.6/11.2 -> 11.2/7.4 us, 13 rows (planes summed by a launch of their own before) 13.5/11.9 -> 12.6/8.0;
// 4096 x 4096 8.0/6.5 -> 8.0/4.7, 12.5/9.4 -> 8.5/5.0; 4096 x 14336 23.7/19.4 -> 23.1/18.0, 25.7/21.6 -> 24.4/18.9.
// With Rotary (qkv) the 16 W rows are eight head-dim indices of a head and their partners half a head dim on: the sums are rounded, rotated
// and go to the qkv row or the cache pages, as gemm_reduce_rope_kernel does it; the first waves take an angle a lane while the first
// stages are on their way.  (One token, 6144 x 4096: 10.4 + 4.9 us as two launches, 12.3 us in one; with all
// angles taken by wave 0 13.4.)
constexpr int kDeep = 4;

struct NoRotary {};
struct Rotary {
    const int32_t *seq_of_token, *pos_of_token, *block_table;
    bf16_t *k_cache, *v_cache;
    RopeTable tab;
    AttnShape sh;
};

template <int S, int XR, class EP>
__global__ __launch_bounds__(64 * S) void gemm_rows16_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                             const bf16_t *__restrict__ R, bf16_t *__restrict__ Y, int rows,
                                                             int N, int K, EP ep) {
    constexpr bool ROTARY = std::is_same_v<EP, Rotary>;
    constexpr int PER_WAVE = S < 4 ? 4 / S : 1;                // angles a lane of the first four waves takes
    __shared__ float2 angle[ROTARY ? 4 : 1][64];               // cosine, sine of row r of wave 0's lanes
    constexpr int LOADS = 2 + XR / 8, STAGE = LOADS * 1024;   // 16 W rows, XR (8 or 16) X rows of 64 k
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];      // a ring of kDeep stages for every wave; in the end the planes' sums
    f32x4(*const planes)[64] = reinterpret_cast<f32x4(*)[64]>(lds);
    const int lane = threadIdx.x & 63, sp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
    int n0 = blockIdx.x * 16, pair = 8;                    // W rows n0 .. n0 + 7 and the eight from n0 + pair on
    int head = 0, i0 = 0;
    if constexpr (ROTARY) {
        const int per_head = ep.sh.head_dim / 16;
        head = blockIdx.x / per_head;
        i0 = blockIdx.x % per_head * 8;
        n0 = head * ep.sh.head_dim + i0;
        pair = ep.sh.head_dim / 2;
    }
    const int Kp = K / S, n_stage = Kp / BK;
    const int rot = (int)(((unsigned)rot_group_of(n0, N) * kRotStep) % (unsigned)n_stage);
    const bf16_t *src[LOADS];                              // 8 rows of a stage by 8 lanes each, the 16-byte columns swizzled with the row
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int row = (j & 1) * 8 + (lane >> 3), col = sp * Kp + ((lane & 7) ^ (row >> 1 & 7)) * 8;
        src[j] = j < 2 ? W + (size_t)(n0 + (row & 7) + (row & 8 ? pair : 0)) * K + col : X + (size_t)min(row, rows - 1) * ldx + col;
    }
    unsigned char *const ring = lds + sp * kDeep * STAGE;
    const unsigned ring0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
    const unsigned adr = ring0 + lr * ROWB + ((lq ^ (lr >> 1 & 7)) << 4);
    const unsigned x_adr = ring0 + 16 * ROWB + (lr % XR) * ROWB + ((lq ^ ((lr % XR) >> 1 & 7)) << 4);      // columns 8..15 of 8 rows: not stored
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    int kst = rot;                                         // next stage to issue
    auto issue = [&](int slot) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + (size_t)kst * BK),
                                             (__attribute__((address_space(3))) void *)(ring + slot * STAGE + j * 1024), 16, 0, 0);
        if (++kst == n_stage) kst = 0;
    };
    auto multiply = [&](auto slot) {                       // a ring is its wave's own: no barrier
        constexpr int AT = decltype(slot)::value * STAGE;
        bf16x8 a0 = lds_read16<AT>(adr), a1 = lds_read16<AT>(adr ^ 64u), b0 = lds_read16<AT>(x_adr), b1 = lds_read16<AT>(x_adr ^ 64u);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a0), "+v"(a1), "+v"(b0), "+v"(b1) : : "memory");
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, acc, 0, 0, 0);
    };
    int pos = 0, seq = 0, page = 0;
    double freq[ROTARY ? PER_WAVE : 1];
    if constexpr (ROTARY)                                  // before the ring's loads: a wait for these is none for those
        if (sp < 4) {
            pos = ep.pos_of_token[min(lr, rows - 1)];
            seq = ep.seq_of_token[min(lr, rows - 1)];
#pragma unroll
            for (int i = 0; i < PER_WAVE; ++i) freq[i] = ep.tab.inv_freq[i0 + 4 * (lq & 1) + sp + i * S];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
    for (int d = 0; d < kDeep; ++d) issue(d);              // a plane has at least 8 stages
    if constexpr (ROTARY)
        if (sp < 4) {
            __builtin_amdgcn_sched_barrier(0);
            if (sp == 0) page = ep.block_table[(size_t)seq * ep.sh.max_pages_per_seq + pos / ep.sh.page_size];
#pragma unroll
            for (int i = 0; i < PER_WAVE; ++i) {
                float s, c;
                rotary_angle(pos, freq[i], s, c);
                angle[sp + i * S][lane] = make_float2(c, s);
            }
        }
    int st = 0;
    for (; st + 2 * kDeep <= n_stage; st += kDeep)
        static_for<0, kDeep>([&](auto d) {
            wait_vmcnt((kDeep - 1) * LOADS);                   // the oldest stage has landed
            multiply(d);
            issue(decltype(d)::value);
        });
    const int left = n_stage - st - kDeep;                 // stages still to issue, less than a ring
    static_for<0, 2 * kDeep - 1>([&](auto d) {
        constexpr int D = decltype(d)::value;
        if (D < left + kDeep) {
            if (D < left) {
                wait_vmcnt((kDeep - 1) * LOADS);
                multiply(std::integral_constant<int, D % kDeep>());
                issue(D % kDeep);
            } else {
                if (D == left) wait_vmcnt(0);
                multiply(std::integral_constant<int, D % kDeep>());
            }
        }
    });
    __syncthreads();                                       // the rings are free
    planes[sp][lane] = acc;
    __syncthreads();
    if (sp != 0 || lr >= rows) return;
    f32x4 o = planes[0][lane];
#pragma unroll
    for (int s = 1; s < S; ++s) o += planes[s][lane];
    if constexpr (ROTARY) {
        const AttnShape &sh = ep.sh;
        const int d = sh.head_dim, at = i0 + 4 * (lq & 1) + (lq >> 1) * pair, slot = pos % sh.page_size;   // lanes 32 on hold the partners
        bf16_t v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = f2bf(o[r]);
            const float mine = bf2f(v[r]), other = __shfl_xor(mine, 32, 64);
            const float2 cs = angle[r][lane];
            if (head < sh.n_q + sh.n_kv) v[r] = f2bf(lq < 2 ? rotated_lo(mine, other, cs.x, cs.y) : rotated_hi(other, mine, cs.x, cs.y));
        }
        if (head < sh.n_q + sh.n_kv) {
            bf16_t *dst = head < sh.n_q ? Y + (size_t)lr * N + head * d : ep.k_cache + (((size_t)page * sh.n_kv + (head - sh.n_q)) * sh.page_size + slot) * d;
            uint2 ov;
            ov.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
            ov.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
            *reinterpret_cast<uint2 *>(dst + at) = ov;
        } else {                                           // v head -> V page [kvh][d][slot]
            bf16_t *vp = ep.v_cache + (((size_t)page * sh.n_kv + (head - sh.n_q - sh.n_kv)) * d + at) * sh.page_size + slot;
#pragma unroll
            for (int r = 0; r < 4; ++r) vp[(size_t)r * sh.page_size] = v[r];
        }
        return;
    }
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

// Where the kernel is taken on the whole chip.  Every workgroup reads all of X for its 16 W rows, so
// with workgroups that are more than the CUs but do not fill them twice the CUs with two set the pace, and two planes of a large
// matrix do not save what that costs.  A layer's step, planes summed by a launch of their own -> in the
// workgroup, us a layer:
//   at most 256 workgroups, or 512 and more: 4096 wide, 14336 MLP, 9 / 13 / 16 rows 117.0 / 119.0 / 117.6 -> 112.5 / 114.3 / 117.2; 3072 x 8192
//     83.3 / 83.8 / 84.6 -> 75.9 / 79.3 / 83.2; 2048 x 5632 65.1 / 66.0 / 66.4 -> 56.3 / 57.7 / 58.9; 3584 x 18944 140.3 / 141.6 / 142.1 -> 136.4 / 139.0
//     / 142.6; 8192 x 28672 359 / 355 / 361 -> 339 / 345 / 351; two planes of 16384 x 2048 (2048 wide, 64-wide heads) 66.7 / 67.5 / 68.9 -> 60.7 / 62.0 / 64.5
//   257 to 511: 5120 x 13824 1 / 4 / 8 / 13 rows 156.8 / 160.5 / 164.0 / 168.6 -> 155.7 / 158.0 / 164.9 / 175.6; 6144 x 16384 209.7 / 214.2 / 215.6 /
//     217.9 -> 208.4 / 212.8 / 217.0 / 223.6; two planes of 15360 x 5120, in the first of these from 13 rows on: 168.6 -> 173.4
// The limit of 6 rows was drawn before the rotary form, which saves a launch more; with it, planes -> workgroup at 7 / 9 / 13 / 16 rows: 4096 wide (qkv
// 6144 x 4096) 124.6 / 125.6 / 129.5 / 130.8 -> 119.0 / 119.8 / 124.7 / 127.1, 5120 x 13824 158.7 / 159.7 / 163.0 / 164.2 -> 149.9 / 153.6 / 160.8 / 164.7,
// 6144 x 16384 214.8 / 216.0 / 220.3 / 222.0 -> 214.9 / 219.4 / 226.7 / 231.2.
bool gemm_rows16_wide_supported(int rows, int N, int K, int S) {
    if (S != 2 && S != 4 && S != 8) return false;
    const int wg = N / 16;
    const bool all = wg <= 256 || (wg >= 512 && (S > 2 || (size_t)N * K <= (size_t)48 << 20));
    return rows <= (all ? 16 : 6);
}

// Where it is taken on any number of CUs: the shapes with the fewest X bytes beside their weights.  (A part of the above.)
bool gemm_rows16_supported(int rows, int N, int K, int S) {
    if (rows > 8 || (S != 2 && S != 4 && S != 8)) return false;
    const int wg = N / 16;
    if (wg <= 256) return S < 8 || rows <= 6 || (long)rows * K <= 8L * N;
    return wg < 512 ? rows <= 2 && K < 2 * N : S > 2 && rows <= 5;
}

// On a partition what a CU gets from its cache bounds the launch rather than memory, and 16 X rows beside 16 W rows are as much again as the
// weights.  The operator, planes summed by a launch of their own -> in the workgroup, us on 64 / 128 / 192 CUs:
//   up to 4 rows: 1 row x 6144 x 4096 43/36/30 -> 37/29/28, x 4096 x 14336 71/51/52 -> 67/48/49, x 8192 x 28672 192/120/122 -> 180/114/101, 4 rows
//     193/121/122 -> 201/124/106
//   8 rows, K < 2 N: x 8192 x 8192 83/61/63 -> 84/60/55; longer: x 3072 x 8192 46/39/33 -> 38/33/29, x 4096 x 14336 73/52/52 -> 79/54/53, x 8192 x 28672
//     196/122/124 -> 227/139/116
//   16 rows: x 3584 x 2560 31/27/27 -> 28/23/23, x 3072 x 8192 46/40/34 -> 42/35/30, x 16384 x 3072 (gate/up) 64/46/45 -> 59/44/42, x 4096 x 14336
//     74/53/53 -> 92/61/60, x 10240 x 8192 92/68/60 -> 115/72/63; where a norm follows, which the launch that sums planes applies too:
//     x 3072 x 3072 36/31/31 -> 34/31/29, x 3584 x 3584 39/33/33 -> 42/35/34, x 4096 x 4096 45/36/37 -> 49/37/38
bool gemm_rows16_taken(int rows, int N, int K, int S, int n_cus, bool norm) {
    if (!gemm_rows16_wide_supported(rows, N, K, S)) return false;
    if (n_cus <= 0 || n_cus >= 256 || rows <= 4 || gemm_rows16_supported(rows, N, K, S)) return true;
    if (rows <= 8 && K < 2 * N) return true;
    return (size_t)N * K <= (size_t)(rows > 8 && norm ? 10 : 48) << 20;
}

// The rotary form: halves of a head in whole eights, and a head's columns in one group of the stage order.
bool gemm_rows16_rope_supported(const AttnShape &sh) {
    return sh.head_dim % 16 == 0 && 128 * kRotGroup % sh.head_dim == 0 && sh.head_dim <= 2 * kMaxHalfDim;
}

namespace {
template <int S, int XR, class EP>
hipError_t launch_rows(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, const EP &ep) {
    constexpr int LDS = S * kDeep * (2 + XR / 8) * 1024;
    static_assert(LDS + 2048 <= 160 * 1024, "the planes' rings do not fit in LDS");
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)gemm_rows16_kernel<S, XR, EP>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_rows16_kernel<S, XR, EP>), dim3(N / 16), dim3(64 * S), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W,
                       (const bf16_t *)R, (bf16_t *)Y, rows, N, K, ep);
    return hipGetLastError();
}

template <class EP>
hipError_t launch_rows_of(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S, const EP &ep) {
    // 8 X rows a stage wherever they are enough: 16 for 6 rows cost 0 to 1 % of a layer's step (5120 wide 141.6 -> 142.5 us a layer), on 64
    // CUs more, with fewer workgroups a CU (2 rows of 3072 wide 111.4 -> 115.8, of 2048 wide 94 -> 103)
    if (rows <= 8)
        return S == 8   ? launch_rows<8, 8>(s, X, ldx, W, R, Y, rows, N, K, ep)
               : S == 4 ? launch_rows<4, 8>(s, X, ldx, W, R, Y, rows, N, K, ep)
                        : launch_rows<2, 8>(s, X, ldx, W, R, Y, rows, N, K, ep);
    return S == 8   ? launch_rows<8, 16>(s, X, ldx, W, R, Y, rows, N, K, ep)
           : S == 4 ? launch_rows<4, 16>(s, X, ldx, W, R, Y, rows, N, K, ep)
                    : launch_rows<2, 16>(s, X, ldx, W, R, Y, rows, N, K, ep);
}
}  // namespace

hipError_t launch_gemm_rows16(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S,
                              const GemmEpilogue *rope) {
    if (!rope) return launch_rows_of(s, X, ldx, W, R, Y, rows, N, K, S, NoRotary{});
    const Rotary ep{rope->seq_of_token, rope->pos_of_token, rope->block_table, (bf16_t *)rope->k_cache, (bf16_t *)rope->v_cache, *rope->rope, *rope->shape};
    return launch_rows_of(s, X, ldx, W, R, Y, rows, N, K, S, ep);
}

}  // namespace dyn
