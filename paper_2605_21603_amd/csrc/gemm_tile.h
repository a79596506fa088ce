// One output tile of a bf16 projection on the matrix cores: the device code that the plain, folded and
// expert-grouped projection kernels share (kernels_gemm.hip, kernels_gemm_wide.hip).
#pragma once
#include "common.h"
#include "kernels.h"

namespace dyn {

// ------------------------------------------------------------------ bf16 MFMA path
// Workgroup = NW waves (4 or 8) on a BN (W rows) x MT (X rows) output tile and one K plane (or,
// INREG, all planes in turn).  What bounds this kernel below a few hundred rows is not the matrix
// cores and not even HBM alone but the L2 -> CU path: every byte of W must cross it once and
// the X tile crosses it once per W tile, so both operands are fetched exactly once per
// workgroup, with fully coalesced 128-byte row segments (8 lanes per row), by direct
// global -> LDS loads (no registers in between) into a ring of NS stage buffers (a stage is
// 64 k); NS - 1 stages are in flight while one is multiplied, tracked with exact vmcnt waits
// and one barrier per stage.  A direct load places lane l's 16 bytes at l * 16 of the wave's
// 1 KB window, so rows sit at a 128-byte pitch; bank conflicts of the MFMA-layout reads
// (lane l: row l%16, 8 consecutive k at 8*(l/16)) are avoided by an XOR swizzle of the
// 16-byte column with bits 1..3 of the row, applied to the global column a lane fetches.
// Waves sit 2 (along X rows; 4 on the tall tiles) x NW/2 (along W rows) on the tile.
// D[i][j]: i = W row (4*(l/16)+r), j = X row (l%16).  Which tile a launch uses is gemm_path's
// decision: 128 x 64|128 with a ring of 4 for few rows, 128 x 256|384|512 for 129..512 rows,
// 256 x 256 for many rows without planes, 256 x 128 with planes folded, 128 x 128|160 with two workgroups
// per CU otherwise.
//
// INREG: one workgroup walks all S planes of its tile and adds the plane sums in registers
// (same order, same bits as the plane buffers + gemm_reduce_kernel) - for many-row launches,
// where there are enough tiles to fill the chip without spreading planes over workgroups and
// the fp32 plane traffic would cost more than the weights.
constexpr int BK = 64, ROWB = BK * 2;
constexpr int kRotGroup = 32, kRotStep = 9;   // stage-order rotation of the bf16 kernel

// Rotation group of the tile at W row n0 of N.  The second half of a wide output counts from its own start: gate and up columns
// that belong together are then summed alike, and a tile may hold both (gemm_gate_fold_kernel).
__device__ __forceinline__ int rot_group_of(int n0, int N) { return (N >= 8192 && N % 512 == 0 && n0 >= N / 2 ? n0 - N / 2 : n0) / 128 / kRotGroup; }

__device__ __forceinline__ void wait_vmcnt(int n) {          // s_waitcnt vmcnt(n) only; n folds to a literal <= 63
    // simm16: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14; expcnt 7 and lgkmcnt 15 = no wait
#define DYN_W(N) case N: __builtin_amdgcn_s_waitcnt(0x0f70 | ((N) & 15) | (((N) >> 4) << 14)); break;
    switch (n) {
        DYN_W(0) DYN_W(2) DYN_W(3) DYN_W(4) DYN_W(5) DYN_W(6) DYN_W(7) DYN_W(8) DYN_W(9) DYN_W(10) DYN_W(12) DYN_W(14) DYN_W(15) DYN_W(16) DYN_W(18) DYN_W(21) DYN_W(24) DYN_W(27) DYN_W(28) DYN_W(32)
        default: __builtin_amdgcn_s_waitcnt(0x0f70); break;       // unknown count: wait for everything
    }
#undef DYN_W
}

// The MFMA as inline assembly, so that the many-row loop's instruction order is the one written down.
// The compiler neither sees the instruction's latency nor orders anything around it: the caller keeps
// dependent uses of an accumulator far apart and waits before reading it as an ordinary register.
__device__ __forceinline__ void mfma_acc(f32x4 &c, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// Waits for the assembly LDS reads into a and b.  A read whose result nobody uses still writes its registers when it
// arrives: they are operands behind the wait, so that none is given to a value (a store's address) before.
template <int NA, int NB>
__device__ __forceinline__ void drain(bf16x8 (&a)[NA], bf16x8 (&b)[NB]) {
    wait_lgkmcnt<0>();
#pragma unroll
    for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(b[i]));
}

// Makes every accumulator an operand here: an ordinary instruction on one stays on its side of this and of the assembly
// around it (across a bare wait the compiler may move it).
template <int NA, int NB>
__device__ __forceinline__ void pin(f32x4 (&acc)[NA][NB]) {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(acc[a][b]));
}
// Waits until the assembly products into acc have left the matrix core.
template <int NA, int NB>
__device__ __forceinline__ void settle(f32x4 (&acc)[NA][NB]) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    pin(acc);
}

// n tiles per band of a launch whose tiles cover the whole depth.  Eight bring an XCD's tiles of every shape
// here to about as many W rows as X rows (32 or 64 tiles run on it at a time).  4096 rows, n-tile order -> bands
// of 8 (4 and 16 lose 1-4 % of it): qkv 252 -> 208, o 183 -> 167, down 528 -> 470, gate/up 763 -> 753 us; 3000 rows: down
// 449 -> 428 us; up to 2112 rows nothing changes.
// A weight matrix of more than 256 MiB does not stay in the last-level cache between two passes over it, and a band
// whose m tiles do not all run at once makes them: there n-tile order is the better one up to 2400 rows, and at every number
// of rows beyond 512 MiB (bands -> n-tile order: 1800 rows x 8192 x 28672 906 -> 805 us, 850 x 27648 x 5120 278 -> 264, 3000 x 57344
// x 8192 2340 -> 2295; against it 2400 x 32768 x 6144 773 -> 787; past the line 4096 x 32768 x 6144 1222 -> 1275, 3600 x 8192 x
// 28672 1677 -> 1850).
constexpr int kBand = 8;
__device__ __forceinline__ int gemm_band(int rows, int N, int K) {
    const size_t w = (size_t)N * K;
    return (w > (size_t)1 << 27 && rows <= 2400) || w > (size_t)1 << 28 ? 1 : kBand;
}
inline int gemm_band_grid(int n_tiles, int m_tiles) { return (n_tiles * m_tiles + 7) / 8 * 8; }

// Tile of workgroup `block` in a launch whose tiles cover the whole depth, in bands.  Workgroup ids are dealt
// round-robin to the 8 XCDs; an XCD takes a contiguous eighth of the tiles in an order that walks bands of
// `band` n tiles down all m tiles, so that what it works on at one time is about as many W rows as X rows.
// (In n-tile order the 32 CUs of an XCD hold two or four n tiles and every m tile: each XCD then reads all
// of X, eight times the matrix in all.)  False: no tile.
__device__ __forceinline__ bool band_tile(int block, int nt, int m_tiles, int band, int &n_tile, int &m_tile) {
    const int v = block / 8, total = nt * m_tiles, chunk = (total + 7) / 8, idx = block % 8 * chunk + v;
    if (v >= chunk || idx >= total) return false;
    const int b = idx / (band * m_tiles), r = idx - b * band * m_tiles, width = min(band, nt - b * band);
    m_tile = r / width;
    n_tile = b * band + r - m_tile * width;
    return true;
}

// The tile of W rows [n_tile * BN, + BN) and X rows [m0, m0 + MT) (below M) over plane sp of S (INREG: all
// planes in turn).  list: X and output rows are list[row] (the X row list[row] / x_div) instead of row.
// planes_only: the plane's fp32 sums go to P whatever S is.  expert: whose weights W are (0: not grouped).  lds: NS * (BN + MT) * ROWB bytes, 1024-byte aligned.
template <int BN, int MT, bool INREG, int NS, bool GATED, int NW, bool PIPE>
__device__ __forceinline__ void gemm_tile(unsigned char *lds, const bf16_t *__restrict__ X, int ldx, const bf16_t *__restrict__ W,
                                          const bf16_t *__restrict__ R, bf16_t *__restrict__ Y, int ldy, float *__restrict__ P,
                                          size_t plane_stride, int M, int N, int K, int S, const int32_t *list, int x_div,
                                          bool planes_only, int n_tile, int sp, int m0, int expert) {
    constexpr int ROWS = BN + MT;                   // rows of a stage buffer: W rows, then X rows
    constexpr int WMW = (NW == 8 && BN < MT) ? 4 : 2;   // waves along m
    constexpr int WNW = NW / WMW, RW = BN / WNW;     // waves along n; W rows per wave column
    constexpr int LPS = ROWS / (NW * 8);            // direct loads per thread and stage (8 rows per wave instruction)
    static_assert(ROWS % (NW * 8) == 0, "the stage's rows must divide among the waves' direct loads");
    constexpr int STAGE = ROWS * ROWB;              // bytes; NS of them form the ring
    constexpr int NA = RW / 16, NB = MT / (16 * WMW);       // 16-row operand tiles per wave
    const int Kp = K / S, kbase = INREG ? 0 : sp * Kp, n_stage = (INREG ? K : Kp) / BK;
    const int plane_stages = Kp / BK;
    const int n0 = n_tile * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4, wn = wave % WNW, wm = wave / WNW;

    // Direct load j of this wave covers stage rows (j * NW + wave) * 8 .. + 8; lane l fetches
    // row + l / 8, global 16-byte column (l % 8) ^ swizzle(row).
    const bf16_t *src[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int row = (j * NW + wave) * 8 + (lane >> 3);
        const int col = (lane & 7) ^ ((row >> 1) & 7);
        if (row < BN) {
            int n = n0 + row;
            if (GATED) {   // stage row = wave half wn, then gate tiles, then up tiles
                const int wn_r = row / RW, in_w = row % RW, up = in_w / (RW / 2);
                n = n_tile * (BN / 2) + wn_r * (RW / 2) + in_w % (RW / 2) + up * (N / 2);
            }
            src[j] = W + (size_t)n * K + kbase + col * 8;
        } else {
            const int mr = min(m0 + row - BN, M - 1);
            src[j] = X + (size_t)(list ? list[mr] / x_div : mr) * ldx + kbase + col * 8;
        }
    }
    // Stage order: the k stages of a plane are visited starting `rot` stages in and wrapping round,
    // with rot a function of the n tile (groups of kRotGroup tiles share one).  Workgroups that run
    // at the same time then read different column offsets of their 8 KB-pitched weight rows, which
    // spreads the requests over the memory channels; tiles of one group keep reading the same X
    // columns together, so X stays shared in L2.  The order depends on (N, K, n tile, expert) only, never
    // on the number of rows, so every schedule adds the same terms in the same order.  Experts rotate one
    // against the next: a down projection's 32 n tiles are one group, and all 256 workgroups of eight experts'
    // read the same columns of rows 28 KB apart (8 experts x 4096 x 14336, two of them per token: 4, 32, 128 tokens 142 -> 128,
    // 180 -> 169, 187 -> 175 us; 256 tokens 194 -> 192; gate/up, seven groups of n tiles, the same within 1 %).
    const int rot_group = !GATED ? rot_group_of(n0, N) : n_tile * (BN / 2) / (INREG ? 128 : 64) / kRotGroup;   // by output column, the same for every tile shape
    const int rot = (int)((unsigned)(rot_group + expert) * kRotStep % (unsigned)plane_stages);
    int iss_w = 0, iss_base = 0;                       // next stage to issue: index inside its plane, plane's first stage
    unsigned char *iss_buf = lds;                      // the pending stage's ring buffer and k offset (issue_begin / issue_one)
    int iss_kst = 0;
    auto issue_begin = [&](int st) {                   // stage st goes into ring buffer st % NS; st ascends by one per call
        iss_buf = lds + (st % NS) * STAGE;
        iss_kst = iss_w + rot;
        if (iss_kst >= plane_stages) iss_kst -= plane_stages;
        iss_kst += iss_base;
        if (++iss_w == plane_stages) { iss_w = 0; iss_base += plane_stages; }
    };
    auto issue_one = [&](int j) {                      // direct load j of the stage begun last
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + (size_t)iss_kst * BK),
                                         (__attribute__((address_space(3))) void *)(iss_buf + (j * NW + wave) * 8 * ROWB),
                                         16, 0, 0);
    };
    auto issue = [&](int st) {                         // all direct loads of stage st
        issue_begin(st);
#pragma unroll
        for (int j = 0; j < LPS; ++j) issue_one(j);
    };

    f32x4 acc[NA][NB], total[INREG ? NA : 1][INREG ? NB : 1];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (INREG) total[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

    // operand read offsets inside a stage buffer (bytes), k-step 0; k-step 1 flips column bit 2
    int a_off[NA], b_off[NB];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int row = wn * RW + a * 16 + lr;
        a_off[a] = row * ROWB + ((lq ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int row = BN + wm * (MT / WMW) + b * 16 + lr;
        b_off[b] = row * ROWB + ((lq ^ ((row >> 1) & 7)) << 4);
    }

    auto fold_plane = [&](int st) {                    // a plane ends: fold its sum into the total, start from zero
        if (INREG && (st + 1) % plane_stages == 0) {
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    total[a][b] += acc[a][b];
                    acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    auto wait_stage = [&](int st) {                    // stage st has landed when at most the loads of the stages issued after it are outstanding
        const int ahead = min(NS - 2, n_stage - 1 - st);
        if (ahead >= 4) wait_vmcnt(4 * LPS);
        else if (ahead == 3) wait_vmcnt(3 * LPS);
        else if (ahead == 2) wait_vmcnt(2 * LPS);
        else if (ahead == 1) wait_vmcnt(LPS);
        else wait_vmcnt(0);
    };

    if constexpr (PIPE) {
        // Many rows: the matrix cores are the bound, and what keeps them waiting is everything that comes
        // in bursts - a block of operand reads before a block of MFMAs, all of a stage's direct loads
        // right after the barrier.  So the loop is laid out by hand, as inline assembly that the
        // compiler neither reorders nor waits for.  A stage is four steps, (k half 0 | 1) x (first |
        // second half of the wave's X tiles).  While the MFMAs of a step issue, the operands of the
        // next step are read from LDS, one read every few MFMAs, across the stage boundary too; the
        // direct loads of the stage that refills this stage's buffer are spread over the last step in
        // the same way.  When a step begins, all that is outstanding is what the previous step read,
        // so lgkmcnt(0) opens it (LDS reads return in order; nothing newer is in flight).  An
        // accumulator is used once per step, so dependent MFMAs are never close.  Every accumulator
        // still receives its k halves and stages in ascending order: the same bits as the plain loop.
        constexpr int H0 = (NB + 1) / 2, H1 = NB - H0, TILE = 16 * ROWB;   // X tiles of the first and of the second half
        bf16x8 a_cur[NA], a_nxt[NA], b_lo[H0], b_hi[H1];
        // Operand tile i of a kind sits 16 rows = TILE bytes after tile 0 (the swizzle depends on the
        // row's low four bits only), so one address per (kind, k half) and an immediate offset do.
        const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
        const unsigned a_adr[2] = {lds0 + (unsigned)a_off[0], lds0 + (unsigned)(a_off[0] ^ 64)};
        const unsigned b_adr[2] = {lds0 + (unsigned)b_off[0], lds0 + (unsigned)(b_off[0] ^ 64)};
        // The MFMAs of av x bv into accumulator columns b0 .. b0 + hb, with item(0) .. item(n_items - 1)
        // spread evenly between them.
        auto step = [&](const bf16x8 (&av)[NA], const auto &bv, auto b0, auto hb, auto n_items, auto &&item) {
            constexpr int B0 = decltype(b0)::value, M = NA * decltype(hb)::value, T = decltype(n_items)::value;
            static_for<0, M>([&](auto i) {
                constexpr int I = decltype(i)::value;
                mfma_acc(acc[I % NA][B0 + I / NA], av[I % NA], bv[I / NA]);
                static_for<0, T>([&](auto k) {
                    if constexpr (decltype(k)::value * M / T == I) item(k);
                });
            });
        };
        const std::integral_constant<int, 0> c0;
        const std::integral_constant<int, H0> ch0;
        const std::integral_constant<int, H1> ch1;
        // All NS ring buffers are filled before the loop; stage st + NS is issued into the buffer of
        // stage st once every wave has taken its last operands out of it.
#pragma unroll
        for (int d = 0; d < NS; ++d)
            if (d < n_stage) issue(d);
        {
            const int ahead = min(NS - 1, n_stage - 1);
            if (ahead >= 3) wait_vmcnt(3 * LPS);
            else if (ahead == 2) wait_vmcnt(2 * LPS);
            else if (ahead == 1) wait_vmcnt(LPS);
            else wait_vmcnt(0);
        }
        __builtin_amdgcn_s_barrier();
        static_for<0, NA>([&](auto k) { a_cur[decltype(k)::value] = lds_read16<decltype(k)::value * TILE>(a_adr[0]); });
        static_for<0, H0>([&](auto k) { b_lo[decltype(k)::value] = lds_read16<decltype(k)::value * TILE>(b_adr[0]); });
        for (int st = 0; st < n_stage; ++st) {
            const unsigned so = (unsigned)(st % NS) * STAGE;
            const unsigned a1 = a_adr[1] + so, b0 = b_adr[0] + so, b1 = b_adr[1] + so;
            wait_lgkmcnt<0>();
            step(a_cur, b_lo, c0, ch0, ch1, [&](auto k) {
                constexpr int K = decltype(k)::value;
                b_hi[K] = lds_read16<(H0 + K) * TILE>(b0);
            });
            wait_lgkmcnt<0>();
            step(a_cur, b_hi, ch0, ch1, std::integral_constant<int, NA + H0>(), [&](auto k) {
                constexpr int K = decltype(k)::value;
                if constexpr (K < NA) a_nxt[K] = lds_read16<K * TILE>(a1);
                else b_lo[K - NA] = lds_read16<(K - NA) * TILE>(b1);
            });
            wait_lgkmcnt<0>();
            step(a_nxt, b_lo, c0, ch0, ch1, [&](auto k) {
                constexpr int K = decltype(k)::value;
                b_hi[K] = lds_read16<(H0 + K) * TILE>(b1);
            });
            wait_lgkmcnt<0>();                     // this wave has taken its last operands out of stage st's buffer
            // One path for every stage, the last included (a second copy of the step's assembly would
            // give each accumulator two definitions to merge at the loop's head): after the last stage
            // the reads fetch operands nobody uses from the other ring buffer, and nothing is issued.
            wait_stage(st + 1);
            __builtin_amdgcn_s_barrier();          // every wave is done with the buffer and sees stage st + 1
            const unsigned no = (unsigned)((st + 1) % NS) * STAGE;
            const unsigned na = a_adr[0] + no, nb = b_adr[0] + no;
            const bool refill = st + NS < n_stage;
            if (refill) issue_begin(st + NS);
            // reads and direct loads alternate while both last, then the rest of the longer list
            constexpr int R = NA + H0, PAIRS = R < LPS ? R : LPS;
            step(a_nxt, b_hi, ch0, ch1, std::integral_constant<int, R + LPS>(), [&](auto k) {
                constexpr int K = decltype(k)::value;
                constexpr bool is_read = K < 2 * PAIRS ? K % 2 == 0 : R > LPS;
                constexpr int idx = K < 2 * PAIRS ? K / 2 : K - PAIRS;
                if constexpr (is_read) {
                    if constexpr (idx < NA) a_cur[idx] = lds_read16<idx * TILE>(na);
                    else b_lo[idx - NA] = lds_read16<(idx - NA) * TILE>(nb);
                } else {
                    if (refill) issue_one(idx);
                }
            });
            if (INREG && (st + 1) % plane_stages == 0) {
                // the compiler does not know that the assembly's results arrive late: the last MFMAs
                // must have left the pipeline before the accumulators are read as ordinary registers,
                // and the cleared accumulators must be written before the next MFMA reads them
                settle(acc);
                fold_plane(st);
                pin(acc);
                asm volatile("s_nop 7" ::: "memory");
            }
        }
        drain(a_cur, b_lo);                        // what the last stage read for a next one
        settle(acc);
    } else {
#pragma unroll
    for (int d = 0; d < NS - 1; ++d)
        if (d < n_stage) issue(d);
    for (int st = 0; st < n_stage; ++st) {
        wait_stage(st);
        // Bare barrier: __syncthreads() would add a fence that drains every outstanding load, which
        // is exactly the prefetch.  The loads of stage st are complete (waited above) and, being
        // direct-to-LDS, visible once complete; the reads of stage st-1 were consumed by MFMAs.
        __builtin_amdgcn_s_barrier();
        if (st + NS - 1 < n_stage) issue(st + NS - 1);
        const unsigned char *buf = lds + (st % NS) * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 av[NA], bv[NB];
#pragma unroll
            for (int a = 0; a < NA; ++a) av[a] = *reinterpret_cast<const bf16x8 *>(buf + (a_off[a] ^ (ks << 6)));
#pragma unroll
            for (int b = 0; b < NB; ++b) bv[b] = *reinterpret_cast<const bf16x8 *>(buf + (b_off[b] ^ (ks << 6)));
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
        fold_plane(st);
    }
    }

    if (GATED) {
#pragma unroll
        for (int a = 0; a < NA / 2; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int m = m0 + wm * (MT / WMW) + b * 16 + lr;
                const int n = n_tile * (BN / 2) + wn * (RW / 2) + a * 16 + 4 * lq;
                if (m >= M) continue;
                const size_t orow = list ? list[m] : m;
                f32x4 g, up;
                if constexpr (INREG) {                 // rounded as the rows of [gate | up] that the planes' sums would store
                    g = total[a][b];
                    up = total[a + NA / 2][b];
#pragma unroll
                    for (int r = 0; r < 4; ++r) { g[r] = bf2f(f2bf(g[r])); up[r] = bf2f(f2bf(up[r])); }
                } else {
                    g = acc[a][b];
                    up = acc[a + NA / 2][b];
                }
                float o[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = g[r] / (1.0f + expf(-g[r])) * up[r];
                u32x2 ov;
                ov[0] = (uint32_t)f2bf(o[0]) | ((uint32_t)f2bf(o[1]) << 16);
                ov[1] = (uint32_t)f2bf(o[2]) | ((uint32_t)f2bf(o[3]) << 16);
                *reinterpret_cast<u32x2 *>(Y + orow * ldy + n) = ov;
            }
        return;
    }
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int m = m0 + wm * (MT / WMW) + b * 16 + lr;
            const int n = n0 + wn * RW + a * 16 + 4 * lq;
            if (m >= M) continue;
            const size_t orow = list ? list[m] : m;
            f32x4 o = INREG ? total[a][b] : acc[a][b];
            if ((S == 1 || INREG) && !planes_only) {
                if (R) {
                    const u32x2 rv = *reinterpret_cast<const u32x2 *>(R + orow * N + n);
                    o[0] += bf2f(rv[0] & 0xffff); o[1] += bf2f(rv[0] >> 16);
                    o[2] += bf2f(rv[1] & 0xffff); o[3] += bf2f(rv[1] >> 16);
                }
                u32x2 ov;
                ov[0] = (uint32_t)f2bf(o[0]) | ((uint32_t)f2bf(o[1]) << 16);
                ov[1] = (uint32_t)f2bf(o[2]) | ((uint32_t)f2bf(o[3]) << 16);
                *reinterpret_cast<u32x2 *>(Y + orow * N + n) = ov;
            } else {
                *reinterpret_cast<f32x4 *>(P + (size_t)sp * plane_stride + orow * N + n) = o;
            }
        }
}

}  // namespace dyn
