// The large projections of the step (bf16, more than a few hundred rows): C[M][N] = A[M][K] *
// W[N][K]^T on tiles of 256 rows x 256 weight rows, with the same epilogues as the small ones.
//
// What bounds them is the clock and the cycles without an MFMA.  The chip holds its clock only as far as the
// energy of the MFMAs, of the LDS reads and of the copies allows (counters at 1024 x 28672 x 4096: 1.94 GHz
// against 2.33 in row kernels, MFMA pipes busy 64 % of the cycles; ablated: MFMAs alone 133 us, with
// their LDS reads 151 us, with the copies 187-198 us).  Hence:
//  - v_mfma_f32_16x16x32_bf16 instead of 32x32x16: the same flops at half the accumulator
//    traffic, 2.05 against 1.80 PFLOP/s in a stream of MFMAs on random operands (2.05 against
//    1.82 GHz); two waves per SIMD, because one wave alone issues it every 19 cycles instead
//    of 16;
//  - 64 x 128 outputs per wave, the fewest LDS bytes per flop that two waves per SIMD allow;
//  - no bubble at a stage's barrier: the fragments of k-step i + 1 are read under the MFMAs of
//    k-step i across stages too, the barrier sits between the stage's two k-steps, and each copy
//    is issued between two MFMAs, with the row offsets in registers and the stage's offset in a
//    scalar (buffer loads to LDS), so a copy costs no vector instruction;
//  - rings of two activation and three weight stages (all 160 KB of LDS): the weights come from
//    HBM or the last-level cache and are requested three stages ahead, the activations sit in L2.
// Together (1024-row gate/up 238 -> 197 us, down 114 -> 94 us, QKV 58 -> 46 us; 2048-row gate/up
// 463 -> 390 us, all with cold weights).
//
// A launch covers its output with 256 x 256 tiles and, where their last round over the 256 CUs
// would be nearly empty, gives some columns or the last rows to a second, smaller tile shape
// (see plan_big).
#include <algorithm>
#include <type_traits>

#include "gemm_common.hpp"
#include "gemm_big.hpp"

namespace orthrus {

namespace {

constexpr int kBK = 64;          // K depth of a stage: one 128-byte line per row
constexpr int kRowBytes = kBK * 2;
constexpr int kWaves = 8;
constexpr int kRingA = 2, kRingB = 3;
constexpr int kLds = 160 * 1024;
constexpr int ring_bytes(int bm, int bn) { return (kRingA * bm + kRingB * bn) * kRowBytes; }
typedef __attribute__((address_space(3))) void lds_void;

#if defined(__HIP_DEVICE_COMPILE__)
// rows of a matrix as a buffer: reads past `bytes` return zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_buffer(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (unsigned)bytes, 0x00020000);
}
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// One BM x BN tile (BN weight rows; SwiGLU: BN / 2 gate and as many up rows) over K stages
// [kt0, kt0 + nk).  WM x WN waves.
template <int BM, int BN, int WM, int WN, bool SW>
__device__ __forceinline__ void big_tile(const GemmArgs &a, char *smem, int m0, int n0, int kt0, int nk, int split,
                                         const BigPlan &p) {
    static_assert(WM * WN == kWaves, "eight waves");
    constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
    constexpr int A_INST = BM / (8 * kWaves), B_INST = BN / (8 * kWaves), INST = A_INST + B_INST;
    constexpr int ABUF = BM * kRowBytes, BBUF = BN * kRowBytes, B_BASE = kRingA * ABUF;
    static_assert(A_INST * 8 * kWaves == BM && B_INST * 8 * kWaves == BN, "copies divide over the waves");
    static_assert(ring_bytes(BM, BN) <= kLds && TM % 16 == 0 && TN % 16 == 0, "tile");
    static_assert(!SW || (FN % 2 == 0 && TN % 16 == 0), "gate and up halves of a wave");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // LDS row r holds 16-byte chunk c at physical chunk c ^ key(r): the 16 lanes of one pass of a
    // fragment read (16 consecutive rows, same chunk) hit 16 distinct 16-byte bank groups.  Lane l
    // of a copy writes row r0 + l / 8 at physical chunk l % 8 and fetches the chunk stored there.
    auto key_of = [](int row) { return (row / 2) % 8; };
    const size_t lda_b = (size_t)a.lda * 2, ldb_b = (size_t)a.K * 2;
    // the tile's rows of A and of the weights as buffers: rows past M or N read as zero
    const int b_cols = SW ? BN / 2 : BN;
    const int b_valid = min(b_cols, a.N - n0);
    const __amdgpu_buffer_rsrc_t ra = rows_buffer((const char *)a.A + (size_t)m0 * lda_b, (size_t)min(BM, a.M - m0) * lda_b);
    // the 64 x 64 blocked copy is padded to whole blocks
    const size_t b_bytes = (size_t)(a.b_blocked ? (b_valid + 63) / 64 * 64 : b_valid) * ldb_b;
    const __amdgpu_buffer_rsrc_t rb0 = rows_buffer((const char *)a.B0 + (size_t)n0 * ldb_b, b_bytes);
    const __amdgpu_buffer_rsrc_t rb1 = rows_buffer((const char *)(SW ? a.B1 : a.B0) + (size_t)n0 * ldb_b, b_bytes);
    const int b_stage = a.b_blocked ? 64 * kRowBytes : kRowBytes;   // bytes between K stages of a weight row
    unsigned avo[A_INST], bvo[B_INST];
#pragma unroll
    for (int i = 0; i < A_INST; ++i) {
        const int row = 8 * (kWaves * i + wave) + lane / 8;
        avo[i] = row * (unsigned)lda_b + ((lane % 8) ^ key_of(row)) * 16;
    }
#pragma unroll
    for (int i = 0; i < B_INST; ++i) {
        const int row = 8 * (kWaves * i + wave) + lane / 8;
        const int src = SW ? row / TN * (TN / 2) + row % (TN / 2) : row;
        const unsigned at = a.b_blocked ? (src / 64 * (a.K / 64) * 64 + src % 64) * kRowBytes : src * (unsigned)ldb_b;
        bvo[i] = at + ((lane % 8) ^ key_of(row)) * 16;
    }
    auto copy_a = [&](int i, int kt, int buf) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(smem + buf * ABUF + (kWaves * i + wave) * 1024), 16,
                                                 avo[i], (kt0 + kt) * kRowBytes, 0, 0);
    };
    auto copy_b = [&](int i, int kt, int buf) {
        // the eight rows of one copy lie in one half of a wave's slice
        const bool up = SW && (8 * (kWaves * i + wave)) % TN >= TN / 2;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(up ? rb1 : rb0,
                                                 (lds_void *)(smem + B_BASE + buf * BBUF + (kWaves * i + wave) * 1024), 16,
                                                 bvo[i], (kt0 + kt) * b_stage, 0, 0);
    };

    // D = W-fragment x A-fragment: lane holds row (lane & 15) of A and four consecutive weight
    // rows 4 (lane / 16) + r, i.e. four consecutive output columns
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int arow = wm * TM + (lane & 15), brow = wn * TN + (lane & 15);
    int aoff[2], boff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int chunk = kk * 4 + (lane >> 4);
        aoff[kk] = arow * kRowBytes + ((chunk ^ key_of(arow)) << 4);
        boff[kk] = B_BASE + brow * kRowBytes + ((chunk ^ key_of(brow)) << 4);
    }
    bf16x8 fa[2][FM], fb[2][FN];
    // fragment i (A fragments first) of k-step kk into register set kk
    auto read1 = [&](int i, int kk, const char *sa, const char *sb) {
        if (i < FM) fa[kk][i] = *(const bf16x8 *)(sa + aoff[kk] + i * 16 * kRowBytes);
        else fb[kk][i - FM] = *(const bf16x8 *)(sb + boff[kk] + (i - FM) * 16 * kRowBytes);
    };
    const bool live = m0 + wm * TM < a.M;   // some row of this wave exists

    // prologue: A stages 0, 1 and weight stages 0, 1, 2 in flight; the first k-step's fragments
#pragma unroll
    for (int st = 0; st < kRingB; ++st) {
        if (st < kRingA) {
#pragma unroll
            for (int i = 0; i < A_INST; ++i) copy_a(i, min(st, nk - 1), st);
        }
#pragma unroll
        for (int i = 0; i < B_INST; ++i) copy_b(i, min(st, nk - 1), st);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm<INST + B_INST>());
    ring_barrier();
    if (live) {
#pragma unroll
        for (int i = 0; i < FM + FN; ++i) read1(i, 0, smem, smem);
    }
    SCHED_FENCE();
    // Stage kt: the MFMAs of its first k-step over the reads of its second; then everyone's copies
    // of stage kt + 1 have landed (only the B_INST copies of weight stage kt + 2 may be left) and
    // everyone has read all of stage kt; then the MFMAs of the second k-step over the first reads of
    // stage kt + 1 and the copies of A stage kt + 2 and weight stage kt + 3 into the buffers just
    // freed.  Copies past the last stage repeat it, so that every iteration issues the same count.
    int ab = 0, bb = 0;
    auto k_loop = [&](auto live_c) {
        constexpr bool L = decltype(live_c)::value;
        for (int kt = 0; kt < nk; ++kt) {
            const int an = ab ^ 1, bn = bb == kRingB - 1 ? 0 : bb + 1;
            const int kta = min(kt + kRingA, nk - 1), ktb = min(kt + kRingB, nk - 1);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                if (kk == 1) {
                    SCHED_FENCE();
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm<B_INST>());
                    ring_barrier();
                    SCHED_FENCE();
                }
                const char *sa = smem + (kk ? an : ab) * ABUF, *sb = smem + (kk ? bn : bb) * BBUF;
                if (!L) {
                    if (kk == 1) {
#pragma unroll
                        for (int i = 0; i < A_INST; ++i) copy_a(i, kta, ab);
#pragma unroll
                        for (int i = 0; i < B_INST; ++i) copy_b(i, ktb, bb);
                    }
                    continue;
                }
#pragma unroll
                for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                    for (int nj = 0; nj < FN; ++nj) {
                        const int i = mi * FN + nj, ni = (mi & 1) ? FN - 1 - nj : nj;
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kk][ni], fa[kk][mi], acc[mi][ni], 0, 0, 0);
                        if (i < FM + FN) read1(i, kk ^ 1, sa, sb);
                        if (kk == 1) {
                            if (i < A_INST) copy_a(i, kta, ab);
                            else if (i < INST) copy_b(i - A_INST, ktb, bb);
                        }
                        SCHED_FENCE();
                    }
            }
            ab = an;
            bb = bn;
        }
    };
    static_assert(FM * FN >= FM + FN && FM * FN >= INST, "an MFMA for every read and copy");
    if (live) k_loop(std::true_type{});
    else k_loop(std::false_type{});
    // the repeated copies of the last iterations still write LDS: drain them before the epilogue
    // reuses the buffers
    __builtin_amdgcn_s_waitcnt(0);

    // LoRA update: acc += U B^T for rows below lora.rows (split 0), 32 columns of U per MFMA step
    // (U as its bf16 rounding plus remainder, two MFMAs), operands straight from global memory; a
    // fragment's 8 columns lie in one adapter's block because ranks are multiples of 16.  The four
    // adapters' pointers are selected in registers: indexed by lane they would be vector loads from
    // the kernel arguments, microseconds each
    if (a.lora.n > 0 && split == 0 && m0 < a.lora.rows) {
        const LoraGemm &L = a.lora;
        const int ldu = L.n * L.r;
        const bf16x8 zero = {};
        auto pick = [](const void *const (&b)[kMaxStepAdapters], int j) {
            static_assert(kMaxStepAdapters == 4, "four pointers");
            return (const bf16 *)(j == 0 ? b[0] : j == 1 ? b[1] : j == 2 ? b[2] : b[3]);
        };
        for (int c0 = 0; c0 < ldu; c0 += 32) {
            const int c = c0 + 8 * (lane >> 4);
            const bool in = c < ldu;
            const int j = in ? c / L.r : 0, kk = in ? c % L.r : 0;
            const bf16 *const b0 = pick(L.b0, j), *const b1 = SW ? pick(L.b1, j) : nullptr;
            bf16x8 ua[FM], ul[FM];
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) {
                const int row = m0 + wm * TM + mi * 16 + (lane & 15);
                const bool ok = in && row < L.rows;
                ua[mi] = ok ? *(const bf16x8 *)((const bf16 *)L.u + (size_t)row * ldu + c) : zero;
                ul[mi] = ok ? *(const bf16x8 *)((const bf16 *)L.u_lo + (size_t)row * ldu + c) : zero;
            }
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
                int col;
                const bf16 *src;
                if constexpr (SW) {
                    col = n0 + wn * (TN / 2) + (ni % (FN / 2)) * 16 + (lane & 15);
                    src = ni < FN / 2 ? b0 : b1;
                } else {
                    col = n0 + wn * TN + ni * 16 + (lane & 15);
                    src = b0;
                }
                const bf16x8 ub = in ? *(const bf16x8 *)(src + (size_t)min(col, a.N - 1) * L.r + kk) : zero;
#pragma unroll
                for (int mi = 0; mi < FM; ++mi) {
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub, ua[mi], acc[mi][ni], 0, 0, 0);
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ub, ul[mi], acc[mi][ni], 0, 0, 0);
                }
            }
        }
    }

    if constexpr (SW) {
        // the bf16 output tile through LDS, so that its rows leave as whole 16-byte pieces
        constexpr int OC = BN / 2, OROW = OC * 2 + 16;
        static_assert(BM * OROW <= ring_bytes(BM, BN), "output tile");
        __syncthreads();
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int ni = 0; ni < FN / 2; ++ni) {
                const f32x4 g = acc[mi][ni], u = acc[mi][ni + FN / 2];
                const int row = wm * TM + mi * 16 + (lane & 15), col = wn * (TN / 2) + ni * 16 + (lane >> 4) * 4;
                *(uint2 *)(smem + row * OROW + col * 2) =
                    uint2{pack_bf16x2(silu(g[0]) * u[0], silu(g[1]) * u[1]), pack_bf16x2(silu(g[2]) * u[2], silu(g[3]) * u[3])};
            }
        __syncthreads();
        constexpr int PPR = OC / 8;
        for (int c = threadIdx.x; c < BM * PPR; c += 64 * kWaves) {
            const int row = c / PPR, part = c % PPR, grow = m0 + row, gcol = n0 + part * 8;
            if (grow < a.M && gcol < a.N)
                *(u32x4 *)((bf16 *)a.out + (size_t)grow * a.ldo + gcol) = *(const u32x4 *)(smem + row * OROW + part * 16);
        }
        return;
    }
    // fp32 rows: stored, added into the residual stream, or this split's share into its own slab.
    // 16-byte stores where the rows allow them
    float *base = p.splits > 1 ? a.partial + (size_t)split * a.split_stride : (float *)a.out;
    const bool add = p.add && p.splits == 1;
    const bool vec = a.ldo % 4 == 0 && (uintptr_t)base % 16 == 0;
#pragma unroll
    for (int mi = 0; mi < FM; ++mi) {
        const int row = m0 + wm * TM + mi * 16 + (lane & 15);
        if (row >= a.M) continue;
        float *o = base + (size_t)row * a.ldo;
#pragma unroll
        for (int ni = 0; ni < FN; ++ni) {
            const int col = n0 + wn * TN + ni * 16 + (lane >> 4) * 4;
            if (vec && col + 3 < a.N) {
                f32x4 v = acc[mi][ni];
                if (add) v += *(const f32x4 *)(o + col);
                *(f32x4 *)(o + col) = v;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (col + r < a.N) o[col + r] = (add ? o[col + r] : 0.f) + acc[mi][ni][r];
            }
        }
    }
}
#endif

// block b of n in XCD-contiguous order: blocks are dealt round-robin to the 8 XCDs, and each
// XCD walks a run of consecutive tiles (row tiles fastest), so re-reads stay inside one L2
__device__ __forceinline__ int xcd_run(int b, int n) {
    const int x = b % 8, q = n / 8, r = n % 8;
    return x * q + min(x, r) + b / 8;
}

// Blocks [0, main * splits): 256 x 256 tiles over row tiles [0, m_main) and the first n_main column
// tiles; the rest: tiles of the second shape over the remaining columns (of every row) or rows.
// MAIN false: the second shape covers everything (and the workgroup takes only its LDS).
template <bool SW, bool MAIN, int BM2, int BN2, int WM2, int WN2>
__global__ __launch_bounds__(64 * kWaves, 1) void gemm_big_kernel(GemmArgs a, BigPlan p) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ __attribute__((aligned(1024))) char smem[MAIN ? kLds : ring_bytes(BM2, BN2)];
    constexpr int C1 = SW ? 128 : 256, C2 = SW ? BN2 / 2 : BN2;
    const int n1 = MAIN ? p.m_main * p.n_main : 0, n2 = p.m_alt * p.n_alt, stages = a.K / kBK;
    int b = blockIdx.x;
    if constexpr (MAIN) {
        if (b < n1 * p.splits) {
            const int split = b / n1, t = xcd_run(b % n1, n1);
            const int kt0 = (int)((long)split * stages / p.splits), kt1 = (int)((long)(split + 1) * stages / p.splits);
            big_tile<256, 256, 4, 2, SW>(a, smem, t % p.m_main * 256, t / p.m_main * C1, kt0, kt1 - kt0, split, p);
            return;
        }
    }
    if constexpr (BM2 > 0) {
        b -= n1 * p.splits;
        const int split = b / n2, t = xcd_run(b % n2, n2);
        const int kt0 = (int)((long)split * stages / p.splits), kt1 = (int)((long)(split + 1) * stages / p.splits);
        big_tile<BM2, BN2, WM2, WN2, SW>(a, smem, p.row_alt + t % p.m_alt * BM2, p.col_alt + t / p.m_alt * C2, kt0, kt1 - kt0,
                                         split, p);
    }
#endif
}

// Tiles of two costs handed in order, the first kind before the second, to 256 CUs as they become free
struct TwoCosts {
    double c1, c2, ratio, inv2;
    TwoCosts(double first, double second) : c1(first), c2(second), ratio(first / second), inv2(1 / second) {}
    // whether the last of n1 and n2 tiles can end before `limit`: n2 tiles' worth of the CUs' time after their
    // first kind
    bool can_end_before(double limit, long n1, long n2) const {
        const long k = n1 % 256;
        const double after_a = (limit - n1 / 256 * c1) * inv2 + 1e-6, after_b = after_a - ratio;
        return after_a > 0 && (long)after_a * (256 - k) + (after_b > 0 ? (long)after_b * k : 0) >= n2;
    }
    // the time of the last
    double makespan(long n1, long n2) const {
        const long k = n1 % 256;
        const double ta = n1 / 256 * c1, tb = ta + c1;   // 256 - k CUs are free at ta, k at tb
        const double end = k ? tb : ta;
        if (n2 == 0) return end;
        // the least time by which the CUs finish n2 more tiles: a tile's end on one of the two groups
        const double average = (n1 * c1 + n2 * c2) * (1.0 / 256);     // load of a CU: no end is before it
        for (long i = std::max(0L, (long)((average - tb) * inv2) - 1);; ++i) {
            // by ta + i c2, by tb + i c2
            const double by_a = i - ratio + 1e-9, by_b = i + ratio + 1e-9;
            if (i * (256 - k) + (by_a > 0 ? (long)by_a * k : 0) >= n2) return std::max(end, ta + i * c2);
            if (k && (long)by_b * (256 - k) + i * k >= n2) return std::max(end, tb + i * c2);
        }
    }
};

// Microseconds of a K stage of a bm x bn tile, and of the rest of a tile (prologue, epilogue).
// Measured over the 7B and the 2048-wide shapes at 160..2048 rows: 256x256 1.45, 256x192 and
// 192x256 1.15-1.18, 192x192 1.0, 128x256 0.95-0.97, 192x128 0.82-0.87, two 128x128 side by side
// on one CU 0.93.
double stage_us(int bm, int bn, int per_cu) { return 0.44 + 0.0155e-3 * bm * bn * per_cu; }
constexpr double kTileUs = 4.0;

struct Shape { int id, bm, bn, per_cu; bool light; };
// shapes that cover an output alone (ids as in launch_shape); per_cu: workgroups whose LDS and
// registers fit one CU; light: at most 120 registers and 112 KB
constexpr Shape kAlone[] = {{4, 192, 256, 1, false}, {5, 192, 192, 1, false}, {6, 192, 128, 1, true}, {7, 128, 256, 1, false},
                            {8, 128, 128, 2, true}, {9, 64, 256, 1, true},  {10, 64, 128, 2, true}};

}  // namespace

// The cover whose estimated length is least.  A round of workgroups lasts as long as its tiles, so
// 256 x 256 tiles win where their rounds are full or nearly so; else their last round goes to
// smaller tiles, or (few rows, where a round of 256 x 256 tiles is never full) one smaller shape
// covers everything.  544 rows of the 7B gate/up: 192x192 130 us, 256x256 154; down, K split
// three ways: 128x128 74 us, 256x256 96.
static BigPlan search_plan(int M, int N, int K, bool swiglu, int splits, bool light) {
    const int C = swiglu ? 128 : 256, f = swiglu ? 2 : 1;
    const int mt = (M + 255) / 256, nt = (N + C - 1) / C;
    const double stages = (double)K / kBK / splits;
    auto tile_us = [&](int bm, int bn) { return stages * stage_us(bm, bn, 1) + kTileUs; };
    const double c256 = tile_us(256, 256);
    BigPlan best;
    best.m_main = mt;
    best.n_main = nt;
    best.splits = splits;
    best.us = light ? 1e30 : TwoCosts(c256, c256).makespan((long)mt * nt * splits, 0);
    auto offer = [&](const BigPlan &p) {
        if (p.us < best.us * 0.98) best = p;
    };
    // the last rows on 128- or 64-row tiles
    const int rem = M % 256;
    if (!light && M > 256 && rem > 0 && rem <= 128) {
        const int bm = rem <= 64 ? 64 : 128;
        BigPlan p;
        p.shape = bm == 64 ? 11 : 1;
        p.m_main = M / 256;
        p.n_main = nt;
        p.m_alt = 1;
        p.n_alt = nt;
        p.row_alt = M - rem;
        p.splits = splits;
        p.us = TwoCosts(c256, tile_us(bm, 256)).makespan((long)p.m_main * nt * splits, (long)nt * splits);
        offer(p);
    }
    // columns past the first j column tiles on 192- or 128-wide tiles
    for (int shape = 2; shape <= 3 && !light; ++shape) {
        const int w = (shape == 2 ? 192 : 128) / f;
        const double inv_w = 1.0 / w;
        const TwoCosts costs(c256, tile_us(256, w * f));
        for (int j = 0; j < nt; ++j) {
            const int n_alt = (int)((N - j * C + w - 0.5) * inv_w);      // the quotient rounded up
            const long n1 = (long)mt * j * splits, n2 = (long)mt * n_alt * splits;
            if (((n1 + 255) >> 8) * c256 >= best.us * 0.98) break;       // the first kind's end alone
            if (!costs.can_end_before(best.us * 0.98, n1, n2)) continue;
            BigPlan p;
            p.us = costs.makespan(n1, n2);
            p.shape = shape;
            p.m_main = mt;
            p.n_main = j;
            p.m_alt = mt;
            p.n_alt = n_alt;
            p.col_alt = j * C;
            p.splits = splits;
            offer(p);
        }
    }
    for (const Shape &sh : kAlone) {
        if (light && !sh.light) continue;
        const int cols = sh.bn / f, m_alt = (M + sh.bm - 1) / sh.bm, n_alt = (N + cols - 1) / cols;
        const unsigned n = (unsigned)m_alt * n_alt * splits, slots = 256u << (sh.per_cu - 1);
        const unsigned left = n & (slots - 1);
        const double full = stages * stage_us(sh.bm, sh.bn, sh.per_cu) + kTileUs;
        BigPlan p;
        p.us = (n >> (7 + sh.per_cu)) * full + (left == 0 ? 0.0 : left <= 256 ? tile_us(sh.bm, sh.bn) : full);
        if (p.us >= best.us * 0.98) continue;
        p.shape = sh.id;
        p.m_alt = m_alt;
        p.n_alt = n_alt;
        p.splits = splits;
        best = p;
    }
    return best;
}

// The search takes up to a microsecond or two; a layer asks for the same covers (about eleven) as the one
// before it, so each thread keeps the last ones it computed (a pure function of the sizes), four to a set.
BigPlan plan_big(int M, int N, int K, bool swiglu, int splits, bool light) {
    struct Entry { int M = 0, N = 0, K = 0, rest = -1; BigPlan plan; };
    constexpr int kSets = 32, kWays = 4;
    static thread_local Entry memo[kSets][kWays];
    static thread_local unsigned char oldest[kSets];
    const int rest = splits * 4 + swiglu * 2 + light;
    uint64_t h = (uint64_t)(unsigned)M << 32 | (unsigned)N;
    for (const uint64_t part : {(uint64_t)(unsigned)K, (uint64_t)(unsigned)rest}) h = ((h ^ h >> 29) + part) * 0x9e3779b97f4a7c15u;
    const int set = (int)(h >> 59);
    static_assert(kSets == 32, "five bits of the hash");
    for (const Entry &e : memo[set])
        if (e.M == M && e.N == N && e.K == K && e.rest == rest) return e.plan;
    Entry &e = memo[set][oldest[set]++ % kWays];
    e = Entry{M, N, K, rest, search_plan(M, N, K, swiglu, splits, light)};
    return e.plan;
}

int big_splits(int M, int N, int K, int max_splits, bool light) {
    int best = 1;
    double best_us = 0.0;
    for (int s = 1; s <= max_splits; ++s) {
        if (s > 1 && (K % kBK || K / s < 512)) continue;
        // the next row kernel reads every slab, at about 4 TB/s
        const double us = plan_big(M, N, K, false, s, light).us + s * ((double)M * N * 4 / 4e6);
        if (s == 1 || us < best_us) { best = s; best_us = us; }
    }
    return best;
}

template <bool SW>
static hipError_t launch_shape(const GemmArgs &a, const BigPlan &p, hipStream_t s) {
    const dim3 grid((p.m_main * p.n_main + p.m_alt * p.n_alt) * p.splits), block(64 * kWaves);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, a, p);
        return hipGetLastError();
    };
    switch (p.shape) {
        case 0: return go(gemm_big_kernel<SW, true, 0, 0, 4, 2>);
        case 1: return go(gemm_big_kernel<SW, true, 128, 256, 2, 4>);
        case 2: return go(gemm_big_kernel<SW, true, 256, 192, 4, 2>);
        case 3: return go(gemm_big_kernel<SW, true, 256, 128, 4, 2>);
        case 4: return go(gemm_big_kernel<SW, false, 192, 256, 2, 4>);
        case 5: return go(gemm_big_kernel<SW, false, 192, 192, 4, 2>);
        case 6: return go(gemm_big_kernel<SW, false, 192, 128, 4, 2>);
        case 7: return go(gemm_big_kernel<SW, false, 128, 256, 2, 4>);
        case 8: return go(gemm_big_kernel<SW, false, 128, 128, 4, 2>);
        case 9: return go(gemm_big_kernel<SW, false, 64, 256, 2, 4>);
        case 10: return go(gemm_big_kernel<SW, false, 64, 128, 2, 4>);
        case 11: return go(gemm_big_kernel<SW, true, 64, 256, 2, 4>);
        default: return hipErrorInvalidValue;
    }
}

// a tile's 256 rows are addressed by 32-bit byte offsets
bool gemm_big_takes(const GemmArgs &a) {
    return a.K > 0 && a.K % kBK == 0 && (size_t)a.lda * 2 * 256 <= 0x7fffffffu && (size_t)a.K * 2 * 256 <= 0x7fffffffu;
}

hipError_t launch_gemm_big(int epi, const GemmArgs &a, const BigPlan &p, hipStream_t s) {
    if (!gemm_big_takes(a) || a.K / kBK < p.splits || (p.splits > 1 && (epi != EPI_ADD_F32 || !a.partial)))
        return hipErrorInvalidValue;
    if (epi == EPI_SWIGLU) return launch_shape<true>(a, p, s);
    if (epi != EPI_STORE_F32 && epi != EPI_ADD_F32) return hipErrorInvalidValue;
    BigPlan q = p;
    q.add = epi == EPI_ADD_F32;
    return launch_shape<false>(a, q, s);
}

}  // namespace orthrus
