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
    if (!band_tile(blockIdx.x, N / 256, (M + 127) / 128, gemm_band(M, N, K), n_tile, m_tile)) return;
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

// The m tile at place `m` of the launch order: an expert's rows are cut into as few m tiles of at most `top` 64s as hold them, the experts
// with the tallest tiles first.  even: an expert's tiles alike, else heights that add up to its rows.  units 0: no tile.  counts: the experts'
// rows, one a lane.  (A lane works its own expert out and counts the tiles before it; expert by expert in scalar code, with a division
// each, a workgroup began 2 us later.)
struct ExpertTile { int units, expert, rows, m0; };
__device__ __forceinline__ ExpertTile expert_tile(int counts, int n_experts, int m, int top, bool even) {
    const int lane = threadIdx.x & 63, all = (counts + 63) / 64, n_m = (all + top - 1) / top, each = max(n_m, 1);
    const int low = even ? ((counts + each - 1) / each + 63) / 64 : all / each, taller = even ? 0 : all - low * each;   // the first `taller` m tiles are 64 rows taller
    const int size = low + (taller > 0);
    int start = 0;                                     // m tiles before this expert's
    for (int e = 0; e < n_experts; ++e) {
        const int n = __builtin_amdgcn_readlane(n_m, e), sz = __builtin_amdgcn_readlane(size, e);
        start += sz > size || (sz == size && e < lane) ? n : 0;
    }
    const unsigned long long mine = __ballot(m >= start && m < start + n_m);
    if (!mine) return ExpertTile{0, 0, 0, 0};
    const int e = __builtin_ctzll(mine), at = m - __builtin_amdgcn_readlane(start, e), rows = __builtin_amdgcn_readlane(counts, e);
    const int lo = __builtin_amdgcn_readlane(low, e), ta = __builtin_amdgcn_readlane(taller, e), m0 = 64 * (at * lo + min(at, ta));
    return ExpertTile{m0 < rows ? lo + (at < ta) : 0, e, rows, m0};   // equal tiles of whole 64s may leave the last one empty
}

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
    int m = v / n_local;                               // place of the m tile in launch order
    const int n_tile = (v - m * n_local) * 8 + u;
    const ExpertTile t = expert_tile(counts, gr.n_groups, m, top, once);
    if (!t.units) return;
    const int32_t *list = gr.lists + (size_t)t.expert * gr.cap;
    const bf16_t *We = W + (size_t)t.expert * gr.w_stride;
#define DYN_BODY(MT, NS) gemm_tile<kExpertsBN, MT, false, NS, GATED, 8, true>(lds, X, ldx, We, nullptr, Y, ldy, P, 0, t.rows, N, K, 1, list, gr.x_div, gr.force_planes, n_tile, 0, t.m0, t.expert)
    if (t.units == 4) DYN_BODY(256, 2);
    else if (t.units == 3) DYN_BODY(192, 2);
    else if (t.units == 2) DYN_BODY(128, 3);
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

// Expert-grouped launch on 128-wide tiles, with or without planes: up to some 200 rows per expert, where the weight stream is the
// bound.  What stands beside a stage's 128 W rows in LDS are the X rows of the tile, and an expert of 40 rows on a 128-row tile brings in
// 88 copies of its last row: the tile's height follows the expert's own count here too (64 to 256 rows, as above), and an
// expert's weights are read once up to 256 rows.  Tallest tiles first, an expert's tiles together; workgroups that share W rows lie a
// multiple of 8 apart (one XCD).  One height for the launch (64, 128 or 256 rows by the average) -> by the count, steps of 8 experts of 4096 x
// 14336, two per token: 100 / 200 / 256 / 300 tokens 655 / 752 / 862 / 965 -> 644 / 744 / 855 / 865 us, prompts of 72 / 312 / 512 / 712 rows 609 / 836 /
// 969 / 1206 -> 596 / 740 / 843 / 1049 us; 64 tokens and fewer are on 64-row tiles either way.
// FEW: no expert has more than 64 rows, one tile each.
constexpr int kExpertsRowsLds = 160 * 1024;           // the bodies' rings: 3 x 48, 4 x 40, 4 x 32, 4 x 24 KB; FEW: the last, one workgroup per CU (two, with rings of three: 1 token's down projection 84 -> 102 us)

template <bool GATED, bool FEW>
__global__ __launch_bounds__(512, 1) void gemm_experts_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                                              bf16_t *__restrict__ Y, int ldy, float *__restrict__ P, size_t plane_stride,
                                                              int N, int K, int S, GemmGroups gr) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int pairs = N / 128 * S, per_m = (pairs + 7) / 8 * 8;      // (n tile, plane) pairs of an m tile
    const int m = blockIdx.x / per_m, ns = blockIdx.x - m * per_m;
    if (ns >= pairs) return;
    ExpertTile t{1, m, FEW ? gr.counts[m] : 0, 0};
    if constexpr (!FEW) t = expert_tile((int)(threadIdx.x & 63) < gr.n_groups ? gr.counts[threadIdx.x & 63] : 0, gr.n_groups, m, 4, false);
    if (!t.units || !t.rows) return;
    const int32_t *list = gr.lists + (size_t)t.expert * gr.cap;
    const bf16_t *We = W + (size_t)t.expert * gr.w_stride;
#define DYN_BODY(MT, NS) gemm_tile<128, MT, false, NS, GATED, 8, (MT >= 256)>(lds, X, ldx, We, nullptr, Y, ldy, P, plane_stride, t.rows, N, K, S, list, gr.x_div, gr.force_planes, ns / S, ns % S, t.m0, t.expert)
    if constexpr (FEW) DYN_BODY(64, 4);
    else if (t.units == 4) DYN_BODY(256, 3);
    else if (t.units == 3) DYN_BODY(192, 4);
    else if (t.units == 2) DYN_BODY(128, 4);
    else DYN_BODY(64, 4);
#undef DYN_BODY
}

namespace {
template <bool GATED, bool FEW>
hipError_t launch_experts(hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, float *P, size_t plane_stride, int N, int K, int S,
                          const GemmGroups &gr) {
    constexpr int LDS = FEW ? 4 * (128 + 64) * ROWB : kExpertsRowsLds;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)gemm_experts_kernel<GATED, FEW>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int m_tiles = FEW ? gr.n_groups : gr.cap / 256 + gr.n_groups;   // at most one m tile of fewer than 256 rows per expert beyond whole ones
    const int grid = (N / 128 * S + 7) / 8 * 8 * m_tiles;
    hipLaunchKernelGGL((gemm_experts_kernel<GATED, FEW>), dim3(grid), dim3(512), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (bf16_t *)Y, ldy, P,
                       plane_stride, N, K, S, gr);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_gemm_experts(bool gated, hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, float *P, size_t plane_stride,
                               int max_rows, int N, int K, int S, const GemmGroups &gr) {
    if (max_rows <= 64)
        return gated ? launch_experts<true, true>(s, X, ldx, W, Y, ldy, P, plane_stride, N, K, S, gr)
                     : launch_experts<false, true>(s, X, ldx, W, Y, ldy, P, plane_stride, N, K, S, gr);
    return gated ? launch_experts<true, false>(s, X, ldx, W, Y, ldy, P, plane_stride, N, K, S, gr)
                 : launch_experts<false, false>(s, X, ldx, W, Y, ldy, P, plane_stride, N, K, S, gr);
}

// Many rows without planes on 256-wide tiles of several heights, tallest first.  256 of them run at a time and a launch of one height is a whole number
// of rounds; heights that add up to the rows let every CU's share be about the same (wide_cut).  Each height's tiles in bands.
template <bool GATED>
__global__ __launch_bounds__(512, 1) void gemm_cut_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W, const bf16_t *__restrict__ R,
                                                          bf16_t *__restrict__ Y, int ldy, int M, int N, int K, WideCut cut) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int nt = N / 256;
    int block = blockIdx.x, size = 4, row0 = 0;
    for (; size >= 1; --size) {
        const int grid = (nt * cut.tiles[size - 1] + 7) / 8 * 8;
        if (block < grid) break;
        block -= grid;
        row0 += cut.tiles[size - 1] * 64 * size;
    }
    int n_tile, m_tile;
    if (size < 1 || !band_tile(block, nt, cut.tiles[size - 1], gemm_band(M, N, K), n_tile, m_tile)) return;
    const int m0 = row0 + m_tile * 64 * size;
    if (m0 >= M) return;
#define DYN_BODY(MT, NS) gemm_tile<256, MT, false, NS, GATED, 8, true>(lds, X, ldx, W, R, Y, ldy, nullptr, 0, M, N, K, 1, nullptr, 1, false, n_tile, 0, m0, 0)
    if (size == 4) DYN_BODY(256, 2);
    else if (size == 3) DYN_BODY(192, 2);
    else if (size == 2) DYN_BODY(128, 3);
    else DYN_BODY(64, 4);
#undef DYN_BODY
}

hipError_t launch_gemm_cut(bool gated, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int ldy, int rows, int N, int K,
                           const WideCut &cut) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_cut_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kExpertsLds);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void *)gemm_cut_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kExpertsLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int grid = 0;
    for (int n : cut.tiles) grid += gemm_band_grid(N / 256, n);
    if (gated)
        hipLaunchKernelGGL(gemm_cut_kernel<true>, dim3(grid), dim3(512), kExpertsLds, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R, (bf16_t *)Y,
                           ldy, rows, N, K, cut);
    else
        hipLaunchKernelGGL(gemm_cut_kernel<false>, dim3(grid), dim3(512), kExpertsLds, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R, (bf16_t *)Y,
                           ldy, rows, N, K, cut);
    return hipGetLastError();
}

// Longest of the 256 CUs' shares when n[i] tiles of cost[i], costs falling, each go to the CU that is free first.
namespace {
// odd: what a CU's last tile takes longer for being alone there, in parts of its cost, where two run side by side.
float longest_share(const int *n, const float *cost, int kinds, float odd = 0.f) {
    struct Level { float load, last; int cus; bool alone; } lv[64];          // CUs by load
    int levels = 1;
    lv[0] = {0.f, 0.f, 256, false};
    for (int k = 0; k < kinds; ++k)
        for (int left = n[k]; left > 0;) {
            int low = 0;
            for (int i = 1; i < levels; ++i)
                if (lv[i].load < lv[low].load) low = i;
            const int take = std::min(left, lv[low].cus);
            left -= take;
            const Level next{lv[low].load + cost[k], cost[k], take, !lv[low].alone};
            lv[low].cus -= take;
            if (lv[low].cus == 0) lv[low] = lv[--levels];
            int same = 0;
            while (same < levels && !(lv[same].load == next.load && lv[same].alone == next.alone)) ++same;
            if (same < levels) lv[same].cus += take;
            else if (levels < 64) lv[levels++] = next;
            else return 1e30f;
        }
    float most = 0.f;
    for (int i = 0; i < levels; ++i) most = std::max(most, lv[i].load + (lv[i].alone ? odd * lv[i].last : 0.f));
    return most;
}
}  // namespace

// The heights with the shortest longest share, tallest tiles first: 192-, 128- and 64-row tiles take 0.80, 0.60 and 0.40 of a 256-row one.  From two
// rounds on and where 4.5 % are to be had: a height's tiles walk all of W once more.  28672 columns 4096 deep, one height (and the last rows' launch) ->
// heights of their own, 800 / 1100 / 1300 / 1700 / 2112 rows 232 / 291 / 334 / 407 / 460 -> 207 / 264 / 301 / 386 / 439 us, steps 546 / 665 / 747 / 888 / 1048 -> 524 /
// 642 / 731 / 869 / 1023; outside the lines 600 rows 186 -> 198, 3000 rows 623 -> 626.  (44 launches of 8 layer widths, 1024 to 8192 deep: 1.07x on average,
// the least 0.98x.)
static const float kWideCost[4] = {1.0f, 0.80f, 0.60f, 0.40f};            // 256, 192, 128, 64 rows
float cut_rounds(const WideCut &cut, int N) {
    const int nt = N / 256, n[4] = {cut.tiles[3] * nt, cut.tiles[2] * nt, cut.tiles[1] * nt, cut.tiles[0] * nt};
    return longest_share(n, kWideCost, 4);
}
bool wide_cut(int rows, int N, float now, WideCut *out) {
    const int units = (rows + 63) / 64;
    if (now < 2.0f) return false;
    float best = now * 0.955f;
    bool found = false;
    for (int n3 = 0; n3 <= std::min(units / 3, 6); ++n3)
        for (int n2 = 0; n2 <= std::min((units - 3 * n3) / 2, 3); ++n2) {
            const int n1 = (units - 3 * n3 - 2 * n2) % 4, n4 = (units - 3 * n3 - 2 * n2) / 4;
            if (n1 > 1) continue;
            const WideCut c{{n1, n2, n3, n4}};
            const float t = cut_rounds(c, N);
            if (t < best) { best = t; *out = c; found = true; }
        }
    return found;
}

// The same for planes folded in registers: 128-wide tiles of 160, 128 and 96 rows, four waves, two workgroups per CU.
__global__ __launch_bounds__(256, 2) void gemm_fold_cut_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W, const bf16_t *__restrict__ R,
                                                               bf16_t *__restrict__ Y, int M, int N, int K, int S, FoldCut cut) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int nt = N / 128;
    int block = blockIdx.x, size = 5, row0 = 0;            // in 32 rows
    for (; size >= 3; --size) {
        const int grid = (nt * cut.tiles[size - 3] + 7) / 8 * 8;
        if (block < grid) break;
        block -= grid;
        row0 += cut.tiles[size - 3] * 32 * size;
    }
    int n_tile, m_tile;
    if (size < 3 || !band_tile(block, nt, cut.tiles[size - 3], gemm_band(M, N, K), n_tile, m_tile)) return;
    const int m0 = row0 + m_tile * 32 * size;
    if (m0 >= M) return;
#define DYN_BODY(MT) gemm_tile<128, MT, true, 2, false, 4, false>(lds, X, ldx, W, R, Y, N, nullptr, 0, M, N, K, S, nullptr, 1, false, n_tile, 0, m0, 0)
    if (size == 5) DYN_BODY(160);
    else if (size == 4) DYN_BODY(128);
    else DYN_BODY(96);
#undef DYN_BODY
}

hipError_t launch_gemm_fold_cut(hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y, int rows, int N, int K, int S,
                                const FoldCut &cut) {
    constexpr int LDS = 2 * (128 + 160) * ROWB;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)gemm_fold_cut_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int grid = 0;
    for (int n : cut.tiles) grid += gemm_band_grid(N / 128, n);
    hipLaunchKernelGGL(gemm_fold_cut_kernel, dim3(grid), dim3(256), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R, (bf16_t *)Y, rows, N, K,
                       S, cut);
    return hipGetLastError();
}

// m tiles of one height or two neighbouring ones, as many as give the shortest longest share.  In rounds of two 128-row tiles a CU: 160-, 128- and 96-row
// tiles take 0.60, 0.50 and 0.43 (a pair's 99 / 83 / 71 us at 4096 x 4096), a CU's odd one 0.6 of its own more, a round of 256 x 128 tiles 0.975.
// One height -> two, 1100 / 1300 / 1700 / 2112 / 2700 rows: qkv (6144 x 4096) 78 / 86 / 131 / 140 / 161 -> 70 / 76 / 121 / 125 / 141 us, o (4096 x 4096) 78 / 74 / 81 /
// 98 / 141 -> 67 / 70 / 74 / 87 / 132, down (4096 x 14336) from 1300 rows 220 / 241 / 290 / 425 -> 213 / 225 / 249 / 412; 1900 and 4096 rows, which fill whole
// rounds, 241 -> 247 and 469 -> 475 with two: left as they are.  (416 launches of 13 layer widths, 1024 to 28672 deep: 1.036x on average; the same
// launch measured in another process differs by up to 4 %.)
// again: what a further height of less than a round costs beside its tiles, in rounds: they walk all of W once more (gemm_fold_cut; all tiles at once
// walk it together).
static const float kFoldCost[3] = {0.60f, 0.50f, 0.43f};
float cut_rounds(const FoldCut &cut, int N) {
    const int nt = N / 128, n[3] = {cut.tiles[2] * nt, cut.tiles[1] * nt, cut.tiles[0] * nt};
    return longest_share(n, kFoldCost, 3, 0.6f);
}
static bool fold_cut(const GemmPath &p, int rows, int N, float again, FoldCut *out) {
    if (p.kind != GEMM_MANY || !p.folded) return false;
    const int nt = N / 128, units = (rows + 31) / 32;
    float best;
    if (p.bn == 256) {
        best = 0.975f * ((p.workgroups + 255) / 256);
    } else {
        const int n[3] = {p.mt == 160 ? p.workgroups : 0, p.mt == 128 ? p.workgroups : 0, 0};
        best = longest_share(n, kFoldCost, 3, 0.6f);
    }
    best *= 0.97f;
    bool found = false;
    for (int k = (units + 4) / 5; k <= (units + 2) / 3; ++k) {
        const FoldCut c = units <= 3 * k   ? FoldCut{{k, 0, 0}}
                          : units <= 4 * k ? FoldCut{{4 * k - units, units - 3 * k, 0}}
                                           : FoldCut{{0, 5 * k - units, units - 4 * k}};
        const int n[3] = {c.tiles[2] * nt, c.tiles[1] * nt, c.tiles[0] * nt}, all = n[0] + n[1] + n[2], last = n[2] ? n[2] : n[1] ? n[1] : n[0];
        const float t = cut_rounds(c, N) + (all > 512 && last < all && last < 512 ? again : 0.f);
        if (t < best) { best = t; *out = c; found = true; }
    }
    return found;
}

bool fold_cut(const GemmPath &p, int rows, int N, FoldCut *out) { return fold_cut(p, rows, N, 0.f, out); }

// For a launch of N x K weights on n_cus CUs (0: all).  Weights of more than 256 MiB do not stay in the last-level cache from one height's tiles to
// the next ones', and less than a round of tiles is no longer than their way from HBM: 2 N K bytes at 4.8 TB/s, beside rounds of 20 us for 1024 of K
// (8192 x 28672, one height / 8 x 128 and 3 x 96 rows / now, 2 x 128 and 11 x 96: 1300 rows 830 / 910 / 797 us, the step 2545 / 2489 / 2375; 1400
// 864 / 895 / 813, 2607 / 2563 / 2468).
bool gemm_fold_cut(const GemmPath &p, int rows, int N, int K, int n_cus, FoldCut *out) {
    if (n_cus > 0 && n_cus < 256) return false;            // (shares of 256 CUs)
    return fold_cut(p, rows, N, (size_t)N * K > (size_t)1 << 27 ? N * (2.f / 4.8e6f) / (20.f / 1024.f) : 0.f, out);
}

// Gate/up with planes, some hundred rows: 64 gate and the matching 64 up columns a workgroup, planes folded in registers and gated, where
// tiles of one height fill the chip once.  What it saves over planes spread over workgroups is their way through memory and the launch that sums
// them (340 rows x 16384 x 2048, two planes: 34.9 + 10.1 us -> 38).  On the hand-laid-out loop from 128 rows a tile (0.5 % of a step).
template <int MT, int NS>
__global__ __launch_bounds__(512, 1) void gemm_gate_fold_kernel(const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W, bf16_t *__restrict__ Y,
                                                                int ldy, int M, int N, int K, int S) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int m_tiles = (M + MT - 1) / MT, u = blockIdx.x % 8, v = blockIdx.x / 8;      // m tiles that share W rows on one XCD
    const int n_tile = v / m_tiles * 8 + u;
    if (n_tile >= N / 128) return;
    gemm_tile<128, MT, true, NS, true, 8, (MT >= 128)>(lds, X, ldx, W, nullptr, Y, ldy, nullptr, 0, M, N, K, S, nullptr, 1, false, n_tile, 0,
                                                       v % m_tiles * MT, 0);
}

// Its tile height for a launch, 0: not taken.  Above 128 rows, while one round of tiles of up to 256 rows holds them; steps, planes over workgroups -> folded:
// 2048 wide, 64-wide heads 130 / 200 / 250 / 340 / 480 rows 94 / 99 / 103 / 150 / 154 -> 90 / 93 / 97 / 143 / 142 us; 2560 wide 130 / 300 / 500 rows 104 / 139 / 172 ->
// 97 / 135 / 163; 1024 wide 130 / 300 / 500 rows 60 / 82 / 89 -> 54 / 73 / 78.  (Gate/up of 11 layer widths, 1024 to 5120 deep, 12 row counts each: 1.016x to 1.220x
// on average.)  What it saves is the same at any depth, and below some height a tile's own time grows faster with it than that of planes on 128 rows: deeper than that
// from 192 rows a tile on (8192 wide, 4096 MLP, tiles of 64 / 128 rows, 160 / 300 rows 78.5 / 100 -> 87.5 / 105 us; 8192 MLP, tiles of 128 / 192 / 256, 129 / 300 / 384 rows
// 0.95x / 1.04x / 1.09x).
int gate_fold_rows(int rows, int N2, int K) {
    if (gemm_split_k(1, N2, K) == 1 || N2 < 8192 || N2 % 512 || rows <= 128 || rows > 512) return 0;
    const int nt = N2 / 128, m_tiles = 256 / nt;           // m tiles of one round
    if (m_tiles < 1) return 0;
    const int mt = ((rows + m_tiles - 1) / m_tiles + 63) / 64 * 64;
    return mt <= 256 && (K <= 5120 || mt >= 192) ? mt : 0;
}

// Its round is several on a partition, where lower tiles, filled less and with less of W behind each X row, cost more than the planes' way through memory:
// below 128 CUs on 256-row tiles alone.  Gate/up, planes over workgroups -> folded, 170 / 360 / 500 rows (tiles of 128, 192, 256), 64 CUs: 2048 wide, 8192 MLP
// 112 / 145 / 178 -> 117 / 150 / 171 us, 2560 wide, 6912 MLP 125 / 162 / 198 -> 131 / 170 / 195; 128 CUs: 78 / 96 / 113 -> 79 / 94 / 105, 84 / 104 / 125 -> 86 / 105 / 118.
bool gate_fold_taken(int rows, int N2, int K, int n_cus) {
    const int mt = gate_fold_rows(rows, N2, K);
    return n_cus <= 0 || n_cus >= 128 ? mt > 0 : mt == 256;
}

hipError_t launch_gemm_gate_fold(hipStream_t s, const void *X, int ldx, const void *W, void *Y, int ldy, int rows, int N2, int K) {
    const int mt = gate_fold_rows(rows, N2, K), S = gemm_split_k(1, N2, K), grid = (N2 / 128 + 7) / 8 * 8 * ((rows + mt - 1) / mt);
#define DYN_GATE_FOLD(MT, NS)                                                                                                                          \
    {                                                                                                                                                  \
        constexpr int LDS = NS * (128 + MT) * ROWB;                                                                                                    \
        static bool attr_set = false;                                                                                                                  \
        if (!attr_set) {                                                                                                                               \
            const hipError_t e = hipFuncSetAttribute((const void *)gemm_gate_fold_kernel<MT, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);    \
            if (e != hipSuccess) return e;                                                                                                             \
            attr_set = true;                                                                                                                           \
        }                                                                                                                                              \
        hipLaunchKernelGGL((gemm_gate_fold_kernel<MT, NS>), dim3(grid), dim3(512), LDS, s, (const bf16_t *)X, ldx, (const bf16_t *)W, (bf16_t *)Y, ldy, \
                           rows, N2, K, S);                                                                                                            \
    }
    if (mt == 256) DYN_GATE_FOLD(256, 3)
    else if (mt == 192) DYN_GATE_FOLD(192, 3)
    else if (mt == 128) DYN_GATE_FOLD(128, 4)
    else DYN_GATE_FOLD(64, 4)
#undef DYN_GATE_FOLD
    return hipGetLastError();
}

}  // namespace dyn
