// Projections: Y[rows, N] = X[rows, K] W[N, K]^T (+ residual).  These are the layer's
// dense contractions (the paper's compute-bound class, Section 2); below roughly 300 rows
// they are in fact bound by streaming W from HBM once, which is what the bf16 kernel is
// shaped for.
//
// Summation order of one output element is a function of (N, K) only: K is cut into
// S = gemm_split_k(N, K) equal planes, each plane is accumulated in ascending k by the same
// 16x16x32 MFMA into an fp32 accumulator starting from zero, and the plane sums are added
// in ascending plane order, then the residual.  Rows never mix, so a row computed in a
// 64-row micro-batch has the same bits as in the merged batch.
#include <cstdlib>

#include <algorithm>
#include <utility>
#include "gemm_tile.h"

namespace dyn {

// ------------------------------------------------------------------ bf16 MFMA path (gemm_tile.h)
constexpr int kBigBN = 128, kBigMT = 128, kBigNS = 2;   // tile and ring depth of the many-row (matrix-core-bound) regime

// The tiles that only GEMM_WIDE and GEMM_MANY launches use walk their tiles in bands; the others spread planes over
// the grid in n-tile order.  (Decided at compile time: as an argument it cost one token's step under 1 %, 128 rows' nothing
// that could be measured.)
constexpr bool gemm_in_bands(int bn, int nw) { return bn == 256 || nw == 4; }

template <int BN, int MT, bool INREG, int NS, bool GATED, int NW>
__global__ __launch_bounds__(NW * 64, (NW == 4 && (BN + MT) * ROWB * NS <= 72 * 1024) ? 2 : 1) void gemm_bf16_kernel(
    const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W, const bf16_t *__restrict__ R,
    bf16_t *__restrict__ Y, int ldy, float *__restrict__ P, size_t plane_stride, int M, int N, int K, int S) {
    constexpr bool BANDS = gemm_in_bands(BN, NW);      // whole-depth tiles of a many-row launch
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int m_tiles = (M + MT - 1) / MT;
    // Workgroup ids are dealt round-robin to the 8 XCDs.
    const int u = blockIdx.x % 8, v = blockIdx.x / 8;
    int m_tile, ns;
    if (BANDS) {
        if (!band_tile(blockIdx.x, N / BN, m_tiles, gemm_band(M, N, K), ns, m_tile)) return;
    } else {
        // Tiles that share W rows (the m tiles of one (n tile, plane)) get ids 8 apart: same XCD,
        // same L2, adjacent in time.
        m_tile = v % m_tiles;
        ns = (v / m_tiles) * 8 + u;
    }
    const int SG = INREG ? 1 : S;                      // planes spread over the grid
    if (!BANDS && ns >= (N / BN) * SG) return;
    gemm_tile<BN, MT, INREG, NS, GATED, NW, (MT >= 256)>(lds, X, ldx, W, R, Y, ldy, P, plane_stride, M, N, K, S, nullptr, 1, false,
                                                         ns / SG, ns % SG, m_tile * MT, 0);   // the hand-laid-out loop pays from 256-row tiles on
                                                                                           // (128 x 128 tiles: 1-2 % slower with it)
}

template <int BN, int MT, bool INREG, int NS, bool GATED = false, int NW = 4>
hipError_t launch_gemm_bf16(int grid, hipStream_t s, const void *X, int ldx, const void *W, const void *R, void *Y,
                            float *partial, size_t plane_stride, int rows, int N, int K, int S, int ldy = 0) {
    constexpr int STAGE = (BN + MT) * ROWB;
    static_assert(NS >= 2 && NS <= 6 && NS * STAGE <= 160 * 1024, "ring does not fit in LDS");
    static bool attr_set = false;                      // above 64 KB of dynamic LDS needs an opt-in, once
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_bf16_kernel<BN, MT, INREG, NS, GATED, NW>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, NS * STAGE);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_bf16_kernel<BN, MT, INREG, NS, GATED, NW>), dim3(grid), dim3(NW * 64), NS * STAGE, s,
                       (const bf16_t *)X, ldx, (const bf16_t *)W, (const bf16_t *)R, (bf16_t *)Y, ldy ? ldy : N, partial,
                       plane_stride, rows, N, K, S);
    return hipGetLastError();
}

// Y = bf16((((P_0 + P_1) + ...) + P_{S-1}) + R), four elements per thread.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const float *__restrict__ P, size_t plane_stride,
                                                          const bf16_t *__restrict__ R, bf16_t *__restrict__ Y,
                                                          size_t n_vec, int S) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += (size_t)gridDim.x * 256) {
        f32x4 o = *reinterpret_cast<const f32x4 *>(P + i * 4);
        for (int s = 1; s < S; ++s) {
            const f32x4 p = *reinterpret_cast<const f32x4 *>(P + (size_t)s * plane_stride + i * 4);
            o[0] += p[0]; o[1] += p[1]; o[2] += p[2]; o[3] += p[3];
        }
        if (R) {
            const uint2 rv = *reinterpret_cast<const uint2 *>(R + i * 4);
            o[0] += bf2f(rv.x & 0xffff); o[1] += bf2f(rv.x >> 16);
            o[2] += bf2f(rv.y & 0xffff); o[3] += bf2f(rv.y >> 16);
        }
        uint2 ov;
        ov.x = (uint32_t)f2bf(o[0]) | ((uint32_t)f2bf(o[1]) << 16);
        ov.y = (uint32_t)f2bf(o[2]) | ((uint32_t)f2bf(o[3]) << 16);
        *reinterpret_cast<uint2 *>(Y + i * 4) = ov;
    }
}

// Matrix-core probe: the main loop of the 256 x 256-tile kernel above without its indexing - eight
// waves, one workgroup per CU, and per stage and wave 64 MFMAs with 24 operand reads from LDS spread
// between them, one barrier, and eight direct loads (64 KB per workgroup) that refill the other
// stage buffer - on operands that are whatever the caller's buffer holds.  Every workgroup walks a
// 256 KB window of the first 16 MiB of the buffer again and again, so the loads hit L2.  What it
// reaches is what the chip gives a loop of this shape with a schedule that has nothing left to
// improve; it depends on the operands (the chip lowers its clock with the activity of its matrix
// pipes: zeros run a third faster than random values), which is why the caller supplies them.
constexpr size_t kMfmaProbeBytes = (size_t)16 << 20;
__global__ __launch_bounds__(512) void mfma_loop_probe_kernel(const unsigned char *__restrict__ src, int n_stages, float *__restrict__ sink) {
    constexpr int STAGE = 65536;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = (lane & 15) + (wave & 3) * 64;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const unsigned addr = lds0 + row * 128 + (((lane >> 4) ^ ((row >> 1) & 7)) << 4);       // conflict-free 16-byte reads, as the projections' operand reads
    const unsigned addr1 = addr ^ 64;                  // k half 1: the other half of the 128-byte row
    const unsigned char *gsrc = src + (size_t)(blockIdx.x % 64) * 262144 + wave * 1024 + lane * 16;
    auto load = [&](int st, int j) {        // 1 KB per wave: part j of stage st's 64 KB; offsets stay below 16 MiB and inside the two stage buffers
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gsrc + ((st * 8 + j) & 31) * 8192),
                                         (__attribute__((address_space(3))) void *)(lds + (st & 1) * STAGE + (j * 8 + wave) * 1024), 16, 0, 0);
    };
    f32x4 acc[1][32];
    bf16x8 fa[2][4], fb[2][8];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[0][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) load(0, j);
    wait_vmcnt(0);
    __builtin_amdgcn_s_barrier();
    static_for<0, 4>([&](auto i) { fa[0][decltype(i)::value] = lds_read16<decltype(i)::value * 2048>(addr); });
    static_for<0, 8>([&](auto i) { fb[0][decltype(i)::value] = lds_read16<16384 + decltype(i)::value * 2048>(addr); });
    for (int st = 0; st < n_stages; ++st) {
        const unsigned so1 = addr1 + (st & 1) * STAGE, sn = addr + ((st + 1) & 1) * STAGE;
        // k half 0: its MFMAs, with the reads of k half 1 and the direct loads of the next stage between them
        wait_lgkmcnt<0>();
        static_for<0, 32>([&](auto i) {
            constexpr int I = decltype(i)::value;
            mfma_acc(acc[0][I], fa[0][I & 3], fb[0][I >> 2]);
            if constexpr (I % 8 == 1 && I / 8 < 4) fa[1][I / 8] = lds_read16<(I / 8) * 2048>(so1);
            if constexpr (I % 4 == 3) fb[1][I / 4] = lds_read16<16384 + (I / 4) * 2048>(so1);
            if constexpr (I % 4 == 2) load(st + 1, I / 4);
        });
        // k half 1; the next stage's buffer is complete once every wave has waited for its loads and passed the barrier
        wait_lgkmcnt<0>();
        wait_vmcnt(0);
        __builtin_amdgcn_s_barrier();
        static_for<0, 32>([&](auto i) {
            constexpr int I = decltype(i)::value;
            mfma_acc(acc[0][I], fa[1][I & 3], fb[1][I >> 2]);
            if constexpr (I % 8 == 1 && I / 8 < 4) fa[0][I / 8] = lds_read16<(I / 8) * 2048>(sn);
            if constexpr (I % 4 == 3) fb[0][I / 4] = lds_read16<16384 + (I / 4) * 2048>(sn);
        });
    }
    drain(fa[0], fb[0]);
    settle(acc);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 32; ++i) v += acc[0][i][0] + acc[0][i][1] + acc[0][i][2] + acc[0][i][3];
    sink[(size_t)blockIdx.x * 512 + tid] = v;        // keeps the products alive
}

size_t mfma_probe_bytes() { return kMfmaProbeBytes; }
double mfma_probe_flops(int n_stages) { return 256.0 * 8 * n_stages * 64 * (16.0 * 16 * 32 * 2); }

hipError_t launch_mfma_probe(const void *buf, int n_stages, float *sink, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)mfma_loop_probe_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * 65536);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(mfma_loop_probe_kernel, dim3(256), dim3(512), 2 * 65536, s, (const unsigned char *)buf, n_stages, sink);
    return hipGetLastError();
}

bool gemm_supported(int dtype, int N, int K) {
    if (dtype == 0) return N > 0 && K > 0;
    return N > 0 && K > 0 && N % 128 == 0 && K % BK == 0;
}

int gemm_split_k(int dtype, int N, int K, int groups) {
    if (dtype == 0) return 1;
    // enough workgroups to occupy 256 CUs twice over, chunks of at least 8 k-steps
    // planes of at least four stages; enough (128-row tile, plane) pairs to occupy the chip
    int S = 1;
    while ((N / 128) * S * std::max(groups, 1) < 192 && K % (S * 2 * BK) == 0 && K / (S * 2) >= 4 * BK * 2) S *= 2;
    return S;
}

namespace {
// Enough 128 x 128 tiles for the many-row regime.  One row of them is not many rows, however wide: to 1.5 rounds of the few-row form's
// workgroups its deeper ring wins, beyond two many-row workgroups a CU do (layers' steps, many -> few, 1 / 16 / 64 / 128 rows: 256 tiles, 6144 wide,
// 220 / 240 / 285 / 353 -> 185 / 202 / 255 / 332 us; 296, 3584 wide, 148 / 163 / 195 / 239 -> 141 / 155 / 195 / 238; 448, 8192 wide, 336 / 376 / 443 / 537
// -> 343 / 383 / 449 / 540).
bool gemm_many_rows(int rows, int N) {
    const int nt = N / kBigBN;
    return N % kBigBN == 0 && nt * ((rows + kBigMT - 1) / kBigMT) >= 256 && (rows > kBigMT || nt >= 384);
}

// 256 x 256 tiles, eight waves of 64 x 128 each: half the operand bytes moved into LDS per FLOP
// of the 128 x 128 tile.  They pay once there are at
// least two m tiles and enough tiles to fill the chip (2112 x 28672 x 4096: 519 -> 432 us; 512
// rows: 164 -> 121 us; 400 rows: 128 us with a 512-row tall tile, 120 us here).  Not for planes
// folded in registers: the second accumulator set does not fit.
bool gemm_wide_tiles(int rows, int N) { return N % 256 == 0 && rows >= 385 && (N / 256) * ((rows + 255) / 256) >= 192; }

// Tile height of the tall-tile path for a launch of `rows` rows with split factor S (0: another path).
int gemm_tall_rows(int rows, int S, int N, int K) {
    if (rows <= 128 || N % 128) return 0;
    if (rows <= 256) return 256;
    if (S == 1) {
        // Without planes because the n tiles alone fill the chip (gate/up): one tall tile up to 384
        // rows (at 264..320 rows 134-137 us with three 128-row tiles, 108-111 us with one of 384),
        // then the 256 x 256 tile where it applies (400..440 rows: 140-144 us -> 120; a 512-row tall
        // tile took 128).  Without planes because the depth is too short to split: as measured before.
        if (N / 128 < 192) return rows > 320 && rows <= 384 ? 384 : 0;
        return rows <= 384 ? 384 : 0;
    }
    if (rows <= 384) return 384;
    if (rows <= 512) return 512;
    if (rows > 1280) return 0;                  // 1025..1280 rows: two 512-row tiles and a launch for the rest (gemm_path)
    // 513..1024 rows with planes.  Folding planes in registers (the many-row path) wins once it is
    // available, unless its tiles fill only one of the two workgroup slots per CU and the plane
    // traffic is small next to the contraction (S / K small: the down projection; 1024 rows: 212 ->
    // 148 us, while qkv and o stay with the folded path: 79 and 66 us against 99 and 81).
    const bool folded_ok = gemm_many_rows(rows, N);
    const bool half_filled = (N / kBigBN) * ((rows + kBigMT - 1) / kBigMT) < 512;
    if (folded_ok && !(half_filled && K >= 1400 * S)) return 0;
    if (rows > 1024) return folded_ok ? 512 : 0;
    return (rows + 383) / 384 <= (rows + 511) / 512 ? 384 : 512;
}

// 256 x 128 tiles for folded planes (kernels_gemm_wide.hip), from the number of 128 x 128 tiles.  They hold the same outputs
// per CU as two 128 x 128 workgroups and run a full round in 0.93-1.0 of the pair's time; but where the last round leaves
// a CU one 128 x 128 workgroup, that one runs alone and ends sooner, and a 256-wide tile does not.  They win where K is long
// or cut into many planes.  Contraction alone, 128 x 128 -> 256 x 128, over 9 layer widths and 50 row counts of 513..4096:
//   K >= 12288, last round at least half filled: -4 to +11 %, +1.5 % on average (4096 rows x 4096 x 14336 449 -> 435 us, 1600
//     rows 236 -> 213)
//   8 planes and more, whole bands, and one round more than half filled or whole rounds: -1.5 to +7.8 % (4096 rows x 4096 x
//     4096 164 -> 157 us, 1450 rows 78 -> 75)
//   the rest: -15 to +3 % (1664 rows x 6144 x 4096 115 -> 130 us, 4096 x 2560 x 1536 56 -> 64, 3000 x 13824 x 2560 235 -> 260)
bool fold_tiles(int tiles, int S, int N, int K) {
    if (N % 256) return false;
    const int last = tiles % 512;                // 0: whole rounds
    if (K >= 12288) return tiles > 256 && (last == 0 || last >= 256);
    return S >= 8 && K >= 4096 && N % (256 * kBand) == 0 && (last == 0 || last >= 496 || (tiles < 512 && last > 256));
}

}  // namespace

GemmPath gemm_path(int dtype, int rows, int N, int K) {
    GemmPath p{};
    p.split = gemm_split_k(dtype, N, K);
    const int S = p.split, nt = N / 128;
    int tall = gemm_tall_rows(rows, S, N, K);
    if (S > 1 && rows > 64 && rows <= 512) {
        // With planes a launch is a whole number of rounds of 256 workgroups, each as long as the 128 + mt rows
        // it brings into LDS per stage take.  One tall tile wins where the (n tile, plane) pairs alone fill the
        // chip; narrow outputs leave CUs idle and want more, lower tiles (operator under events, 340 rows: 3072 x 2048, 96
        // pairs, 384 -> 256 rows 29.3 -> 25.6 us, 2048 x 2048, 64 pairs, 384 -> 128 rows 27.6 -> 18.9 us; 200 rows: 22.0 -> 19.1, 20.5 -> 15.3 us).
        long best = 0;
        for (int mt : {512, 384, 256, 128, 64}) {
            if (mt > 128 && rows <= mt / 2) continue;            // taller than the rows need
            const long cost = ((long)nt * S * ((rows + mt - 1) / mt) + 255) / 256 * (128 + mt);
            if (!best || cost < best) { best = cost; tall = mt; }
        }
        if (tall <= 128) {
            p.kind = GEMM_FEW; p.bn = 128; p.mt = tall;
            p.workgroups = nt * S * ((rows + tall - 1) / tall);
            p.resident = 256;
            return p;
        }
    }
    if (tall) {
        // 129..512 rows (up to 1024 with planes, see gemm_tall_rows): tall tiles.  Two to four
        // 128-row tiles would move every weight byte into LDS that many times; one tile of 256, 384
        // or 512 rows (eight waves 4 x 2) moves it once: qkv / o / gate-up / down at 256 rows 41 / 34 /
        // 90 / 60 us -> 33 / 28 / 79 / 48 us, o and down at 512 rows 61 / 112 -> 45 / 84 us.  Same planes,
        // same k order, so the same bits.  Without planes the 256 x 256 tile takes over at 385 rows.
        p.kind = GEMM_TALL; p.bn = 128; p.mt = tall;
        // past 1024 rows (the down projection only, see gemm_tall_rows): a third 512-row tile would
        // be a third round of workgroups for at most 256 rows, so those run as a launch of their own
        // (1032 / 1280 rows: 209 / 211 us with planes folded in registers, ~170 this way)
        if (rows > 1024) { p.tail_rows = rows - 1024; rows = 1024; }
        p.workgroups = nt * S * ((rows + tall - 1) / tall);
        p.resident = 256;
        return p;
    }
    // Many-row launches are bound by the matrix cores: enough tiles without spreading planes over
    // workgroups, a shallow ring and two workgroups per CU so that one multiplies while the other
    // waits at its barrier.  Few-row launches are bound by memory: deep ring, one workgroup per CU.
    if (gemm_many_rows(rows, N)) {
        p.folded = S > 1;
        if (S == 1 && gemm_wide_tiles(rows, N)) {
            p.kind = GEMM_WIDE; p.bn = 256; p.mt = 256;
            // 256 tiles run at a time.  When the last m tile alone costs a further round of them,
            // its rows go to a launch of their own on 128-row-wide tiles (one round of N / 128
            // workgroups, shorter than a round here): 520..768 rows of gate/up 208-223 us -> ~180.
            const int m = (rows + 255) / 256, per_m = N / 256;
            if (m >= 3 && (per_m * m + 255) / 256 > (per_m * (m - 1) + 255) / 256) p.tail_rows = rows - 256 * (m - 1);
            p.workgroups = per_m * (p.tail_rows ? m - 1 : m);
            p.resident = 256;
            return p;
        }
        // Tile height: two 4-wave workgroups fit a CU, so 512 tiles run at a time and the launch takes
        // ceil(tiles / 512) rounds of a duration that grows with the tile height.  A taller
        // tile that saves a round wins (2112 rows x 4096 columns: 544 tiles of 128 rows need
        // two rounds, 448 tiles of 160 rows one): a round of 160-row tiles takes 1.29 of one of 128-row tiles (x 14336 deep at
        // 2112 rows: 283 us, one round, against 407, two).  The summation order of an output element does not depend on the tile.
        const long rounds128 = (nt * ((rows + 127) / 128) + 511) / 512, rounds160 = (nt * ((rows + 159) / 160) + 511) / 512;
        p.kind = GEMM_MANY; p.bn = 128; p.mt = rounds160 * 129 < rounds128 * 100 ? 160 : 128;
        p.resident = 512;
        if (p.folded && p.mt == 128 && fold_tiles(nt * ((rows + 127) / 128), S, N, K)) { p.bn = 256; p.resident = 256; }
        p.workgroups = (N / p.bn) * ((rows + p.mt - 1) / p.mt);
        return p;
    }
    p.kind = GEMM_FEW; p.bn = 128; p.mt = rows <= 64 ? 64 : 128;
    p.workgroups = nt * S * ((rows + p.mt - 1) / p.mt);
    p.resident = 256;
    return p;
}

// A GEMM_WIDE launch on tiles of several heights, where that is the faster way; else p as it is: rounds of 256 tiles, and the last rows' launch
// at what it takes beside a round (gate/up of 28672 columns, 64 / 128 / 256 rows: 48 / 60 / 76 us, a round 122).
bool gemm_cut(const GemmPath &p, int rows, int N, int n_cus, WideCut *cut) {
    if (p.kind != GEMM_WIDE || (n_cus > 0 && n_cus < 256)) return false;      // (shares of 256 CUs)
    const float tail = p.tail_rows == 0 ? 0.f : p.tail_rows <= 64 ? 0.40f : p.tail_rows <= 128 ? 0.49f : 0.62f;
    return wide_cut(rows, N, (p.workgroups + 255) / 256 + tail, cut);
}

bool gemm_uses_plane_buffer(int dtype, int rows, int N, int K) {
    if (dtype == 0 || rows <= 0) return false;
    const GemmPath p = gemm_path(dtype, rows, N, K);
    return p.split > 1 && !p.folded;
}

namespace {
// The operator that follows the projection, as a kernel of its own on the rows the projection wrote.
hipError_t run_epilogue(int dtype, const GemmEpilogue &ep, void *Y, int rows, int N, hipStream_t s) {
    if (ep.kind == GemmEpilogue::NORM) return launch_rmsnorm(dtype, Y, ep.g, ep.h_out, ep.ld_h, rows, N, ep.eps, s, &ep.route);
    if (ep.kind == GemmEpilogue::ROPE)
        return launch_rope_kv(dtype, Y, ep.seq_of_token, ep.pos_of_token, ep.block_table, ep.k_cache, ep.v_cache, *ep.rope, *ep.shape, rows,
                              ep.long_rows, s);
    if (ep.kind == GemmEpilogue::GATE) return launch_silu_mul(dtype, Y, ep.h_out, ep.ld_h, rows, N / 2, s);
    return hipSuccess;
}

GemmEpilogue epilogue_at(const GemmEpilogue &ep, int dtype, int row, int N) {      // the same epilogue for rows starting `row` rows in
    GemmEpilogue e = ep;
    const size_t es = dtype == 0 ? 4 : 2;
    if (e.kind == GemmEpilogue::NORM || e.kind == GemmEpilogue::GATE) e.h_out = (char *)e.h_out + (size_t)row * e.ld_h * es;
    if (e.route.w_router) { e.route.sel += (size_t)row * e.route.top_k; e.route.wgt += (size_t)row * e.route.top_k; }
    if (e.kind == GemmEpilogue::ROPE) { e.seq_of_token += row; e.pos_of_token += row; }
    (void)N;
    return e;
}
}  // namespace

hipError_t launch_gemm(int dtype, const void *X, int ldx, const void *W, const void *R, void *Y, float *partial,
                       size_t plane_stride, int rows, int N, int K, hipStream_t s, hipEvent_t mid, const GemmEpilogue *ep, int n_cus,
                       const GemmNorm &norm) {
    if (rows <= 0) return hipSuccess;
    const GemmGroups none{};
    const bool has_ep = ep && ep->kind != GemmEpilogue::NONE;
    if (dtype == 0) {
        const bool rope = has_ep && ep->kind == GemmEpilogue::ROPE && !R && gemm_f32_rope_supported(X, ldx, W, rows, N, K, *ep->shape);
        hipError_t e0 = rope ? launch_gemm_f32_rope(X, ldx, W, Y, rows, N, K, norm, *ep, s) : launch_gemm_f32(X, ldx, W, R, Y, rows, N, K, none, s);
        if (e0 == hipSuccess && mid) e0 = hipEventRecord(mid, s);
        if (e0 == hipSuccess && has_ep && !rope) e0 = run_epilogue(dtype, *ep, Y, rows, N, s);
        return e0;
    }
    const GemmPath p = gemm_path(dtype, rows, N, K);
    WideCut cut;
    if (gemm_cut(p, rows, N, n_cus, &cut)) {
        hipError_t ec = launch_gemm_cut(false, s, X, ldx, W, R, Y, N, rows, N, K, cut);
        if (ec == hipSuccess && mid) ec = hipEventRecord(mid, s);
        if (ec == hipSuccess && has_ep) ec = run_epilogue(dtype, *ep, Y, rows, N, s);
        return ec;
    }
    if (p.tail_rows) {         // the last rows in a launch of their own (own tiles, own planes and reduce)
        const int head = rows - p.tail_rows;
        GemmEpilogue tail_ep;
        if (has_ep) tail_ep = epilogue_at(*ep, dtype, head, N);
        hipError_t et = launch_gemm(dtype, (const bf16_t *)X + (size_t)head * ldx, ldx, W, R ? (const bf16_t *)R + (size_t)head * N : nullptr,
                                    (bf16_t *)Y + (size_t)head * N, partial ? partial + (size_t)head * N : nullptr, plane_stride,
                                    p.tail_rows, N, K, s, nullptr, has_ep ? &tail_ep : nullptr, n_cus);
        if (et != hipSuccess) return et;
        rows = head;
    }
    if (gemm_rows16_taken(rows, N, K, p.split, n_cus, has_ep && ep->kind == GemmEpilogue::NORM)) {
        const bool rope = has_ep && ep->kind == GemmEpilogue::ROPE && !R && gemm_rows16_rope_supported(*ep->shape);
        hipError_t er = launch_gemm_rows16(s, X, ldx, W, R, Y, rows, N, K, p.split, rope ? ep : nullptr);
        if (er == hipSuccess && mid) er = hipEventRecord(mid, s);
        if (er == hipSuccess && has_ep && !rope) er = run_epilogue(dtype, *ep, Y, rows, N, s);
        return er;
    }
    const int S = p.split, m_tiles = (rows + p.mt - 1) / p.mt;
    // workgroup ids are dealt to the 8 XCDs in turn: tiles, or (n tile, plane) pairs, are padded to a multiple of 8
    const int grid = p.kind == GEMM_WIDE || p.kind == GEMM_MANY ? gemm_band_grid(N / p.bn, m_tiles) : (((N / p.bn) * (p.folded ? 1 : S) + 7) / 8) * 8 * m_tiles;
#define DYN_GEMM(BN, MT, INREG, NS, NW) \
    launch_gemm_bf16<BN, MT, INREG, NS, false, NW>(grid, s, X, ldx, W, R, Y, partial, plane_stride, rows, N, K, S)
    hipError_t e;
    FoldCut fold;
    if (gemm_fold_cut(p, rows, N, K, n_cus, &fold)) e = launch_gemm_fold_cut(s, X, ldx, W, R, Y, rows, N, K, S, fold);
    else if (p.kind == GEMM_TALL) e = p.mt == 256 ? DYN_GEMM(128, 256, false, 3, 8) : p.mt == 384 ? DYN_GEMM(128, 384, false, 2, 8) : DYN_GEMM(128, 512, false, 2, 8);
    else if (p.kind == GEMM_WIDE) e = DYN_GEMM(256, 256, false, 2, 8);
    else if (p.kind == GEMM_MANY && p.bn == 256) e = launch_gemm_fold(grid, s, X, ldx, W, R, Y, rows, N, K, S);
    else if (p.kind == GEMM_MANY && p.mt == 160) e = p.folded ? DYN_GEMM(kBigBN, 160, true, kBigNS, 4) : DYN_GEMM(kBigBN, 160, false, kBigNS, 4);
    else if (p.kind == GEMM_MANY) e = p.folded ? DYN_GEMM(kBigBN, kBigMT, true, kBigNS, 4) : DYN_GEMM(kBigBN, kBigMT, false, kBigNS, 4);
    else e = p.mt == 64 ? DYN_GEMM(128, 64, false, 4, 8) : DYN_GEMM(128, 128, false, 4, 8);
#undef DYN_GEMM
    if (e == hipSuccess && mid) e = hipEventRecord(mid, s);
    if (e != hipSuccess) return e;
    if (S == 1 || p.folded) return has_ep ? run_epilogue(dtype, *ep, Y, rows, N, s) : hipSuccess;
    // the planes are summed in plane order, with the residual; where an operator follows on the same rows, by its fused form
    if (has_ep && ep->kind == GemmEpilogue::NORM && N % 8 == 0)
        return launch_reduce_norm(partial, plane_stride, S, R, Y, ep->g, ep->h_out, ep->ld_h, rows, N, ep->eps, s, &ep->route);
    if (has_ep && ep->kind == GemmEpilogue::ROPE && !R && reduce_rope_supported(dtype, *ep->shape))
        return launch_reduce_rope(partial, plane_stride, S, Y, ep->seq_of_token, ep->pos_of_token, ep->block_table, ep->k_cache,
                                  ep->v_cache, *ep->rope, *ep->shape, rows, s);
    if (has_ep && ep->kind == GemmEpilogue::GATE) return launch_reduce_gate(partial, plane_stride, S, ep->h_out, ep->ld_h, rows, N / 2, s);
    const size_t n_vec = (size_t)rows * N / 4;
    const int blocks = (int)((n_vec + 255) / 256 < 2048 ? (n_vec + 255) / 256 : 2048);
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3(blocks), dim3(256), 0, s, partial, plane_stride, (const bf16_t *)R,
                       (bf16_t *)Y, n_vec, S);
    e = hipGetLastError();
    if (e == hipSuccess && has_ep) e = run_epilogue(dtype, *ep, Y, rows, N, s);
    return e;
}

namespace {
// Whether an expert-grouped launch is on 256-wide tiles, from the average number of rows per group (the lists' capacity holds every row
// once).  To about 200 rows per expert the weight stream is the bound; beyond, a 256 x 256 tile's half the operand bytes per FLOP are
// (eight experts' gate/up at 1024 / 2048 tokens: 989 / 1847 us with 128-row tiles, 751 / 1231).  The 256-wide tile has no planes.
bool gemm_experts_on_wide(const GemmGroups &gr, int N, int S) { return S == 1 && N % 256 == 0 && gr.cap / std::max(gr.n_groups, 1) > 200; }
}  // namespace

bool gemm_norm_in_supported(int dtype, int rows, int N, int K, int n_cus) { return dtype == 0 && gemm_f32_norm_supported(rows, N, K, n_cus); }

bool gemm_gated_supported(int dtype, int N2, int K, bool experts) {
    return dtype == 1 ? gemm_split_k(dtype, N2, K) == 1 : !experts && gemm_f32_gated_supported(N2, K);
}

// act[rows or listed rows, N2/2] = silu(X Wg^T) * (X Wu^T) with W = [gate rows; up rows] ([N2, K]),
// output row pitch ldy.  Plain (gr.n_groups = 0: X, Y offset to the dispatch) or expert-grouped.
hipError_t launch_gemm_gated(int dtype, const void *X, int ldx, const void *W, void *Y, int ldy, const GemmGroups &gr, int max_rows,
                             int N2, int K, hipStream_t s, hipEvent_t mid, const GemmNorm &norm, int n_cus) {
    if (max_rows <= 0) return hipSuccess;
    hipError_t e;
    if (dtype == 0) {
        e = launch_gemm_f32_gated(X, ldx, W, Y, ldy, max_rows, N2, K, norm, s);
        return e == hipSuccess && mid ? hipEventRecord(mid, s) : e;
    }
#define DYN_GATED(BN, MT, NS, NW) \
    launch_gemm_bf16<BN, MT, false, NS, true, NW>(grid, s, X, ldx, W, nullptr, Y, nullptr, 0, max_rows, N2, K, 1, ldy)
    if (gr.n_groups) {
        e = gemm_experts_on_wide(gr, N2, 1) ? launch_gemm_experts_wide(true, s, X, ldx, W, Y, ldy, nullptr, N2, K, gr)
                                            : launch_gemm_experts(true, s, X, ldx, W, Y, ldy, nullptr, 0, max_rows, N2, K, 1, gr);
    } else if (gemm_split_k(1, N2, K) > 1) {
        e = launch_gemm_gate_fold(s, X, ldx, W, Y, ldy, max_rows, N2, K);
    } else {
        const GemmPath p = gemm_path(1, max_rows, N2, K);          // split factor 1: no planes on any path
        WideCut cut;
        if (gemm_cut(p, max_rows, N2, n_cus, &cut)) {
            e = launch_gemm_cut(true, s, X, ldx, W, nullptr, Y, ldy, max_rows, N2, K, cut);
            return e == hipSuccess && mid ? hipEventRecord(mid, s) : e;
        }
        if (p.tail_rows) {     // the last rows in a launch of their own (never a wide one: at most 256 rows)
            const int head = max_rows - p.tail_rows;
            e = launch_gemm_gated(dtype, (const bf16_t *)X + (size_t)head * ldx, ldx, W, (bf16_t *)Y + (size_t)head * ldy, ldy, gr,
                                  p.tail_rows, N2, K, s, nullptr, norm, n_cus);
            if (e != hipSuccess) return e;
            max_rows = head;
        }
        const int mt = p.kind == GEMM_MANY ? kBigMT : p.mt;    // the gated many-row kernel has 128-row tiles only
        const int m_tiles = (max_rows + mt - 1) / mt;
        const int grid = p.kind == GEMM_WIDE || p.kind == GEMM_MANY ? gemm_band_grid(N2 / p.bn, m_tiles) : ((N2 / p.bn + 7) / 8) * 8 * m_tiles;
        if (p.kind == GEMM_TALL) e = p.mt == 256 ? DYN_GATED(128, 256, 3, 8) : DYN_GATED(128, 384, 2, 8);
        else if (p.kind == GEMM_WIDE) e = DYN_GATED(256, 256, 2, 8);
        else if (p.kind == GEMM_MANY) e = DYN_GATED(kBigBN, kBigMT, kBigNS, 4);
        else e = p.mt == 64 ? DYN_GATED(128, 64, 4, 8) : DYN_GATED(128, 128, 4, 8);
    }
#undef DYN_GATED
    if (e == hipSuccess && mid) e = hipEventRecord(mid, s);
    return e;
}

// Expert-grouped form: group e multiplies the rows named by its list with its own weight
// matrix W + e * w_stride.  max_rows bounds any group's row count (it sizes the grid; tiles
// past a group's count exit at once).  X, Y and partial are indexed by the lists' row ids (not
// relative to the dispatch); the dispatch's output rows are row0 .. row0 + n_rows - 1.  With
// gr.force_planes the fp32 plane sums go to `partial` for every split factor, including 1, and
// nothing is written to Y.
hipError_t launch_gemm_grouped(int dtype, const void *X, int ldx, const void *W, void *Y, float *partial,
                               size_t plane_stride, const GemmGroups &gr, int max_rows, int row0, int n_rows, int N, int K,
                               hipStream_t s, hipEvent_t mid) {
    if (max_rows <= 0 || gr.n_groups <= 0) return hipSuccess;
    if (dtype == 0) {
        hipError_t e0 = launch_gemm_f32(X, ldx, W, nullptr, gr.force_planes ? partial : Y, max_rows, N, K, gr, s);
        if (e0 == hipSuccess && mid) e0 = hipEventRecord(mid, s);
        return e0;
    }
    const int S = gemm_split_k(dtype, N, K, gr.n_groups);
    hipError_t e = gemm_experts_on_wide(gr, N, S) ? launch_gemm_experts_wide(false, s, X, ldx, W, Y, N, partial, N, K, gr)
                                                  : launch_gemm_experts(false, s, X, ldx, W, Y, N, partial, plane_stride, max_rows, N, K, S, gr);
    if (e == hipSuccess && mid) e = hipEventRecord(mid, s);
    if (e != hipSuccess || S == 1 || gr.force_planes) return e;
    // output rows row0 .. row0 + n_rows - 1 are exactly the rows the groups wrote
    const size_t n_vec = (size_t)n_rows * N / 4;
    const int blocks = (int)((n_vec + 255) / 256 < 2048 ? (n_vec + 255) / 256 : 2048);
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3(blocks), dim3(256), 0, s, partial + (size_t)row0 * N, plane_stride,
                       (const bf16_t *)nullptr, (bf16_t *)Y + (size_t)row0 * N, n_vec, S);
    return hipGetLastError();
}

}  // namespace dyn
