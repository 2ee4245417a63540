// Dense projections of the step: C[M][N] = A[M][K] * W[N][K]^T over the concatenated token
// batch (QKV, attention output, gate/up, down, LM head), with fused epilogues, and the choice of
// kernel per shape (dispatch_bf16; above 128 rows mostly gemm_big.hip).
//
// bf16 path, kernel of this file: CDNA4 MFMA v_mfma_f32_32x32x16_bf16, WM x WN wave64s per workgroup, K staged 64
// elements at a time through two LDS buffers filled by direct global->LDS copies
// (global_load_lds_dwordx4, no register staging), so each K stage costs one barrier.  LDS rows
// are 128 B; 16-byte chunks are XOR-swizzled by row so the per-lane 16-byte operand reads of
// one MFMA hit distinct banks (the copies pick their source chunk to land in swizzled order).
// Tiles are mapped to blocks so that consecutive tiles of one weight column block land on
// the same XCD (blocks are dealt round-robin to the 8 XCDs), which keeps re-reads of a
// weight tile inside one L2.
// fp32 path: v_mfma_f32_32x32x2_f32, one 32x32 tile per workgroup, or two by two where many outputs fill
// the chip with them (exact checks, small models).
#include <algorithm>
#include <type_traits>

#include "gemm_big.hpp"
#include "gemm_common.hpp"
#include "orthrus.h"

namespace orthrus {

namespace {

constexpr int BK = 64;

// STREAM_B: the launch has one row tile, so each weight byte is read exactly once; its copies
// are non-temporal (LM head 64 x 32000 x 4096 in the step: 66 -> 56 us)
template <int BM, int BN, int WM, int WN, int EPI, int BKS, int STAGES, int BSTAGES, bool STREAM_B>
__global__ __launch_bounds__(64 * WM * WN, 1) void gemm_bf16_kernel(GemmArgs a) {
    constexpr int NW = WM * WN;               // waves per workgroup
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int ROWB = BKS * 2;             // bytes of one LDS row (BKS bf16 of K)
    constexpr int CHUNKS = ROWB / 16;         // 16-byte chunks per row
    constexpr int RPI = 1024 / ROWB;          // rows moved by one wave copy instruction (1 KiB)
    constexpr int RP256 = 256 / ROWB;         // rows per 256 bytes (one pass of the 64 LDS banks)
    // global -> LDS copies of one K stage
    constexpr int A_INST = BM / (RPI * NW), B_INST = BN / (RPI * NW);
    constexpr int INST = A_INST + B_INST;     // copy instructions per wave per stage
    constexpr int KSTEPS = BKS / 16;
    // separate rings for A (STAGES buffers of BM rows) and B (BSTAGES buffers of BN rows): the
    // weight operand may prefetch deeper than the activations within the same LDS budget
    constexpr int RING_BYTES = STAGES * BM * ROWB + BSTAGES * BN * ROWB;
    // the shallower ring's copies are issued first in every iteration; vector-memory operations
    // complete in order, so iteration kt may leave these many copies of this wave in flight when
    // it waits for its stage kt (the deeper ring's copies issued after the shallower's stage kt)
    constexpr int SD = STAGES < BSTAGES ? STAGES : BSTAGES, SDD = STAGES < BSTAGES ? BSTAGES : STAGES;
    constexpr int DEEP_INST = STAGES < BSTAGES ? B_INST : A_INST;
    constexpr int IN_FLIGHT = (SD - 2) * INST + (SDD > SD ? DEEP_INST : 0);
    static_assert(A_INST * RPI * NW == BM && B_INST * RPI * NW == BN, "copy split");
    static_assert(FM >= 1 && FN >= 1 && (EPI != EPI_SWIGLU || FN % 2 == 0), "tile shape");
    static_assert(SD >= 2 && IN_FLIGHT < 64, "pipeline depth");
    __shared__ __attribute__((aligned(1024))) char smem[RING_BYTES];
    char *const smem_b = smem + STAGES * BM * ROWB;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int mt = (a.M + BM - 1) / BM;
    constexpr int COLS_ = EPI == EPI_SWIGLU ? BN / 2 : BN;
    const int tiles = mt * ((a.N + COLS_ - 1) / COLS_);
    const int splits = gridDim.x / tiles;          // split-K factor (1 = whole K per tile)
    const int split = blockIdx.x / tiles;
    const int b = blockIdx.x % tiles;
    const int t = (tiles % 8 == 0) ? (b % 8) * (tiles / 8) + b / 8 : b;
    const int n_tile = t / mt, m_tile = t % mt;
    const int m0 = m_tile * BM;
    constexpr int COLS = EPI == EPI_SWIGLU ? BN / 2 : BN;  // output columns per tile
    const int n0 = n_tile * COLS;

    // LDS row r holds 16-byte chunk c at physical position c ^ key(r), key(r) = (r / RP256) %
    // CHUNKS, so the 16 lanes of one pass of a fragment read (16 consecutive rows, same chunk)
    // hit 16 distinct 16-byte bank groups.  Lane `lane` of copy instruction i of this wave
    // writes LDS bytes base + 16 * lane, i.e. row r0 + lane / CHUNKS at physical chunk
    // lane % CHUNKS (r0 = RPI * (NW i + wave)); it fetches the logical chunk stored there.
    auto key_of = [](int row) { return (row / RP256) % CHUNKS; };
    const size_t lda_b = (size_t)a.lda * 2, ldb_b = (size_t)a.K * 2;
    const char *a_src[A_INST];
    const char *b_src[B_INST];
#pragma unroll
    for (int i = 0; i < A_INST; ++i) {
        const int row = RPI * (NW * i + wave) + lane / CHUNKS;
        const int chunk = (lane % CHUNKS) ^ key_of(row);
        a_src[i] = (const char *)a.A + (size_t)min(m0 + row, a.M - 1) * lda_b + chunk * 16;
    }
#pragma unroll
    for (int i = 0; i < B_INST; ++i) {
        const int r = RPI * (NW * i + wave) + lane / CHUNKS;
        const int chunk = (lane % CHUNKS) ^ key_of(BM + r);
        int grow;
        const char *src = (const char *)a.B0;
        if (EPI == EPI_SWIGLU) {
            const int slice = r / TN, j = r % TN;
            const int half = j / (TN / 2), k = j % (TN / 2);
            if (half) src = (const char *)a.B1;
            grow = n0 + slice * (TN / 2) + k;
        } else {
            grow = n0 + r;
        }
        const int gn = min(grow, a.N - 1);
        b_src[i] = a.b_blocked ? src + ((size_t)(gn / 64) * (a.K / 64) * 64 + gn % 64) * ROWB + chunk * 16
                               : src + (size_t)gn * ldb_b + chunk * 16;
    }
    const size_t b_stage = a.b_blocked ? 64 * ROWB : ROWB;   // bytes between k-stages of a B row
    // this wave's copies of K stage kt of A (into A buffer buf) and of B (into B buffer buf)
    auto copy_a = [&](int kt, int buf) {
        const size_t kb = (size_t)kt * ROWB;
#pragma unroll
        for (int j = 0; j < A_INST; ++j)
            copy16_to_lds(a_src[j] + kb, smem + buf * BM * ROWB + (NW * j + wave) * 1024);
    };
    auto copy_b = [&](int kt, int buf) {
        const size_t kb = (size_t)kt * b_stage;
#pragma unroll
        for (int j = 0; j < B_INST; ++j)
            copy16_to_lds<STREAM_B ? kNonTemporal : 0>(b_src[j] + kb, smem_b + buf * BN * ROWB + (NW * j + wave) * 1024);
    };
    // iteration i's copies: A stage i + STAGES - 1 and B stage i + BSTAGES - 1 (the shallower
    // ring first).  Past the last stage they repeat it into the buffer just freed, which nobody
    // reads, so every iteration issues the same count and the wait bound stays exact.
    auto issue = [&](int i, int kt0, int nk) {
        const int sa = i + STAGES - 1, sb = i + BSTAGES - 1;
        if (STAGES <= BSTAGES) {
            if (sa >= 0) copy_a(kt0 + min(sa, nk - 1), sa % STAGES);
            if (sb >= 0) copy_b(kt0 + min(sb, nk - 1), sb % BSTAGES);
        } else {
            if (sb >= 0) copy_b(kt0 + min(sb, nk - 1), sb % BSTAGES);
            if (sa >= 0) copy_a(kt0 + min(sa, nk - 1), sa % STAGES);
        }
    };

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // fragment rows of this lane; the swizzle key is the same for every 32-row fragment of the
    // lane (32 rows span a whole number of 256-byte passes), so offsets differ by constants
    // (B rows keep the swizzle key of row BM + r, as the copies above write them)
    const int arow = wm * TM + (lane & 31), brow = wn * TN + (lane & 31);
    const int akey = key_of(arow), bkey = key_of(BM + brow);
    bf16x8 fa[2][FM], fb[2][FN];
    auto lds_frag = [&](const char *sa, const char *sb, int kk, int buf) {
        const int chk = kk * 2 + (lane >> 5);
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
            fa[buf][mi] = *(const bf16x8 *)(sa + (arow + mi * 32) * ROWB + ((chk ^ akey) << 4));
#pragma unroll
        for (int ni = 0; ni < FN; ++ni)
            fb[buf][ni] = *(const bf16x8 *)(sb + (brow + ni * 32) * ROWB + ((chk ^ bkey) << 4));
    };

    // Rings of LDS stages: the copies of A stage kt + STAGES - 1 and B stage kt + BSTAGES - 1
    // are issued while stage kt is computed.  Iteration kt: wait for this wave's copies of
    // stage kt (later ones stay in flight), barrier (everyone's copies landed; everyone
    // finished reading the buffers about to be refilled), issue, then the MFMAs of stage kt
    // with the next k-step's fragments read under the current k-step's.  (Spreading the copies
    // between the MFMAs, or L2 prefetches further ahead, measured slower on MI355X.)
    constexpr int NMF = FM * FN, NFR = FM + FN;
    // this split's stages: [kt0, kt0 + nk), the K stages dealt as evenly as the count allows
    const int nk_all = a.K / BKS;
    const int kt0 = split * nk_all / splits;
    const int nk = (split + 1) * nk_all / splits - kt0;
    for (int i = -(SDD - 1); i < 0; ++i) issue(i, kt0, nk);
    // A wave whose rows all lie past M (in the last row tile, when M leaves it partly empty)
    // issues its share of the copies and takes every barrier but reads no fragments and issues
    // no MFMA: its accumulators stay zero and its rows are never stored (1088 rows on 256-row
    // tiles: 1.18x -> 1.06x executed / algorithmic flops).
    auto k_loop = [&](auto live) {
        for (int kt = 0; kt < nk; ++kt) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm<IN_FLIGHT>());
            ring_barrier();
            issue(kt, kt0, nk);
            if constexpr (decltype(live)::value) {
                // the compute phase at raised wave priority: where both waves of a SIMD have an
                // instruction ready, the one feeding the MFMA pipe issues first (1024-row gate/up
                // alone 211.9 -> 204.0 us, down 107.6 -> 103.8 us; raising the copy phase
                // instead, or both at different levels, measured equal or slower)
                __builtin_amdgcn_s_setprio(1);
                const char *sa = smem + (kt % STAGES) * BM * ROWB, *sb = smem_b + (kt % BSTAGES) * BN * ROWB;
                lds_frag(sa, sb, 0, 0);
#pragma unroll
                for (int kk = 0; kk < KSTEPS; ++kk) {
                    if (kk + 1 < KSTEPS) lds_frag(sa, sb, kk + 1, (kk + 1) & 1);
#pragma unroll
                    for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                        for (int ni = 0; ni < FN; ++ni)
                            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][mi], fb[kk & 1][ni],
                                                                                  acc[mi][ni], 0, 0, 0);
                }
                // schedule: DS_READ=0x100, MFMA=0x008
                __builtin_amdgcn_sched_group_barrier(0x100, NFR, 0);
#pragma unroll
                for (int kk = 0; kk < KSTEPS; ++kk) {
#pragma unroll
                    for (int i = 0; i < NMF; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        if (kk + 1 < KSTEPS && i < NFR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                }
                __builtin_amdgcn_s_setprio(0);
            }
        }
    };
    // the wave's row range is the same for all its lanes; taking lane 0's answer makes the
    // branch scalar, so each wave runs exactly one of the two loops (equal barrier counts)
    if (__builtin_amdgcn_readfirstlane(m0 + wm * TM < a.M ? 1 : 0)) k_loop(std::true_type{});
    else k_loop(std::false_type{});
    // the repeated copies of the last iterations still write LDS: drain them before the
    // epilogues reuse the stage buffers
    __builtin_amdgcn_s_waitcnt(0);

    // LoRA update: acc += U B^T for the launch's rows below lora.rows (split 0 of a split-K
    // launch), 16 columns of U per MFMA step (U as its bf16 rounding plus remainder, two MFMAs),
    // operands straight from global memory in the same fragment layout as the main loop (rows
    // of U and of B are contiguous in the rank)
    if (a.lora.n > 0 && split == 0 && m0 < a.lora.rows) {
        const LoraGemm &L = a.lora;
        const int ldu = L.n * L.r;
        const bf16x8 zero = {};
        for (int c0 = 0; c0 < ldu; c0 += 16) {
            const int j = c0 / L.r, kk = c0 % L.r + 8 * (lane >> 5);
            bf16x8 ua[FM], ul[FM], ub[FN];
#pragma unroll
            for (int mi = 0; mi < FM; ++mi) {
                const int row = m0 + wm * TM + mi * 32 + (lane & 31);
                const size_t off = (size_t)row * ldu + c0 + 8 * (lane >> 5);
                ua[mi] = row < L.rows ? *(const bf16x8 *)((const bf16 *)L.u + off) : zero;
                ul[mi] = row < L.rows ? *(const bf16x8 *)((const bf16 *)L.u_lo + off) : zero;
            }
#pragma unroll
            for (int ni = 0; ni < FN; ++ni) {
                int col;
                const bf16 *src;
                if constexpr (EPI == EPI_SWIGLU) {
                    col = n0 + wn * (TN / 2) + (ni % (FN / 2)) * 32 + (lane & 31);
                    src = (const bf16 *)(ni < FN / 2 ? L.b0[j] : L.b1[j]);
                } else {
                    col = n0 + wn * TN + ni * 32 + (lane & 31);
                    src = (const bf16 *)L.b0[j];
                }
                ub[ni] = *(const bf16x8 *)(src + (size_t)min(col, a.N - 1) * L.r + kk);
            }
#pragma unroll
            for (int mi = 0; mi < FM; ++mi)
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) {
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ua[mi], ub[ni], acc[mi][ni], 0, 0, 0);
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ul[mi], ub[ni], acc[mi][ni], 0, 0, 0);
                }
        }
    }

    if constexpr (EPI == EPI_SWIGLU) {
        // The MFMA layout leaves each lane one column of 16 rows per fragment, i.e. 2-byte
        // stores per output.  Instead the BM x BN/2 bf16 output tile is staged through the
        // idle stage buffers and written back as whole 16-byte pieces of its rows.
        constexpr int OC = BN / 2;                 // output columns of the tile
        constexpr int OROW = OC * 2 + 16;          // padded LDS row: rows 4 apart differ by 16 banks
        static_assert(BM * OROW <= RING_BYTES, "output tile fits the stage buffers");
        __syncthreads();                           // every wave is done with the stage buffers
#pragma unroll
        for (int mi = 0; mi < FM; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm * TM + mi * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
#pragma unroll
                for (int ni = 0; ni < FN / 2; ++ni) {
                    const int col = wn * (TN / 2) + ni * 32 + (lane & 31);
                    *(bf16 *)(smem + row * OROW + col * 2) = (bf16)(silu(acc[mi][ni][r]) * acc[mi][ni + FN / 2][r]);
                }
            }
        __syncthreads();
        constexpr int PPR = OC / 8;                // 16-byte pieces per row
        for (int c = tid; c < BM * PPR; c += 64 * NW) {
            const int row = c / PPR, part = c % PPR;
            const int grow = m0 + row, gcol = n0 + part * 8;
            if (grow < a.M && gcol < a.N)
                *(u32x4 *)((bf16 *)a.out + (size_t)grow * a.ldo + gcol) = *(const u32x4 *)(smem + row * OROW + part * 16);
        }
        return;
    }

    // epilogue: lane holds column (lane & 31) of each 32x32 tile, rows 8*(r/4) + 4*(lane/32) + r%4
#pragma unroll
    for (int mi = 0; mi < FM; ++mi) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * TM + mi * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (row >= a.M) continue;
            if (EPI == EPI_SWIGLU) {
                bf16 *o = (bf16 *)a.out + (size_t)row * a.ldo;
#pragma unroll
                for (int ni = 0; ni < FN / 2; ++ni) {
                    const int col = n0 + wn * (TN / 2) + ni * 32 + (lane & 31);
                    if (col < a.N) o[col] = from_f32<bf16>(silu(acc[mi][ni][r]) * acc[mi][ni + FN / 2][r]);
                }
            } else if (splits > 1) {
                // split-K: this split's share goes to its own fp32 slab; the row's consumer adds
                // the slabs to the residual stream in split order
                float *o = a.partial + (size_t)split * a.split_stride + (size_t)row * a.ldo;
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) {
                    const int col = n0 + wn * TN + ni * 32 + (lane & 31);
                    if (col < a.N) o[col] = acc[mi][ni][r];
                }
            } else {
                float *o = (float *)a.out + (size_t)row * a.ldo;
#pragma unroll
                for (int ni = 0; ni < FN; ++ni) {
                    const int col = n0 + wn * TN + ni * 32 + (lane & 31);
                    if (col >= a.N) continue;
                    if (EPI == EPI_ADD_F32) o[col] += acc[mi][ni][r];
                    else o[col] = acc[mi][ni][r];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ fp32 reference-grade path
// 32 x 32 outputs per workgroup on v_mfma_f32_32x32x2_f32 (fp32 products and sums), its eight waves
// splitting K in runs of eight, their partial tiles summed through LDS in wave order.  Operands come
// straight from global memory: a lane reads four consecutive k of its row and half (16 bytes) and
// feeds them to four MFMAs, both operands in the same order.  The fp32 models are the small ones
// (K <= 1024, a few hundred rows), where a call lasts as long as one workgroup's chain: short
// K runs and many workgroups count (260 x 256 outputs, K 256 and 1024: 69 us on average on 64x64
// LDS tiles of scalar FMAs with 20 workgroups, 8.9 us with 72 of these).
// TWO: two row tiles by two weight tiles (or by gate and up) per wave, where the outputs fill the chip with
// them (run_f32).  What bounds one tile there is the rate of its loads, which touch 32 rows for 1 KB: two
// need half the loads per MFMA (7B shape, 512 rows: gate/up 2333 -> 1683 us, QKV 520 -> 371; 2048 rows: 9160 ->
// 6416, 2021 -> 1400; LM head of 256 rows 1688 -> 976).  Each output is summed in the same order either way.
constexpr int kF32Waves = 8, kF32Run = 4;   // waves; 16-byte loads per operand and register set
template <int EPI, bool TWO>
__global__ __launch_bounds__(64 * kF32Waves) void gemm_f32_kernel(GemmArgs a) {
    constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;       // weight matrices
    constexpr int RM = TWO ? 2 : 1, RN = TWO && NB == 1 ? 2 : 1, RB = NB * RN;
    __shared__ float red[kF32Waves][NB][32 * 33];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // one tile: weight tiles fastest; two: row tiles fastest, so that large weights leave HBM once
    const int m0 = (TWO ? blockIdx.x : blockIdx.y) * (32 * RM), n0 = (TWO ? blockIdx.y : blockIdx.x) * (32 * RN), half = lane >> 5;
    const int chunks = a.K / 8;                       // runs of 8 k: 4 for each half of the wave
    const int c0 = wave * chunks / kF32Waves, c1 = (wave + 1) * chunks / kF32Waves;
    const float *pa[RM], *pb[RB];
#pragma unroll
    for (int i = 0; i < RM; ++i) pa[i] = (const float *)a.A + (size_t)min(m0 + 32 * i + (lane & 31), a.M - 1) * a.lda + 4 * half;
#pragma unroll
    for (int j = 0; j < RB; ++j)
        pb[j] = (const float *)(NB == 2 && j ? a.B1 : a.B0) + (size_t)min(n0 + (NB == 2 ? 0 : 32 * j) + (lane & 31), a.N - 1) * a.K + 4 * half;
    f32x16 acc[RM][RB];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    f32x4 va[2][RM][kF32Run], vb[2][RB][kF32Run];
    // runs [c, c + kF32Run) of this wave into set s, as many as it has
    auto load = [&](int c, int s) {
#pragma unroll
        for (int k = 0; k < kF32Run; ++k) {
            if (c + k >= c1) break;
#pragma unroll
            for (int i = 0; i < RM; ++i) va[s][i][k] = *(const f32x4 *)(pa[i] + 8 * (c + k));
#pragma unroll
            for (int j = 0; j < RB; ++j) vb[s][j][k] = *(const f32x4 *)(pb[j] + 8 * (c + k));
        }
    };
    auto mul = [&](int c, int s) {
#pragma unroll
        for (int k = 0; k < kF32Run; ++k) {
            if (c + k >= c1) break;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[s][i][k][e], vb[s][j][k][e], acc[i][j], 0, 0, 0);
        }
    };
    load(c0, 0);
    for (int c = c0; c < c1; c += 2 * kF32Run) {
        load(c + kF32Run, 1);
        mul(c, 0);
        load(c + 2 * kF32Run, 0);
        mul(c + kF32Run, 1);
    }
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            if (i + j > 0) __syncthreads();           // the tile before has been read
            // lane holds column lane % 32, rows 8 (e / 4) + 4 (lane / 32) + e % 4
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    red[wave][x][((e >> 2) * 8 + half * 4 + (e & 3)) * 33 + (lane & 31)] = acc[i][NB == 2 ? x : j][e];
            __syncthreads();
            for (int o = tid; o < 32 * 32; o += 64 * kF32Waves) {
                const int r = o / 32, c = o % 32, row = m0 + 32 * i + r, col = n0 + 32 * j + c;
                if (row >= a.M || col >= a.N) continue;
                float v[NB];
#pragma unroll
                for (int x = 0; x < NB; ++x) {
                    v[x] = red[0][x][r * 33 + c];
#pragma unroll
                    for (int w = 1; w < kF32Waves; ++w) v[x] += red[w][x][r * 33 + c];
                }
                if (a.lora.n > 0 && row < a.lora.rows) {      // LoRA update U B^T
                    const LoraGemm &L = a.lora;
                    const int ldu = L.n * L.r;
                    const float *u = (const float *)L.u + (size_t)row * ldu;
#pragma unroll
                    for (int x = 0; x < NB; ++x) {
                        float d = 0.f;
                        for (int k = 0; k < ldu; ++k)
                            d = fmaf(u[k], ((const float *)(x ? L.b1 : L.b0)[k / L.r])[(size_t)col * L.r + k % L.r], d);
                        v[x] += d;
                    }
                }
                float *out = (float *)a.out + (size_t)row * a.ldo + col;
                if (EPI == EPI_SWIGLU) *out = silu(v[0]) * v[NB - 1];
                else if (EPI == EPI_ADD_F32) *out += v[0];
                else *out = v[0];
            }
        }
}

// Two tiles where their rounds of workgroups over the chip take less time: a round of them lasts as long as
// 3.1 of one tile each, 1.6 for gate/up (K 4096: 134 us against 43, 137 against 84).  256 rows by 4096, one
// round against four: 173 -> 136 us; 160 by 6144, two against four: 179 stays, 240 on two.
template <int EPI>
hipError_t run_f32(const GemmArgs &a, hipStream_t s) {
    constexpr bool sw = EPI == EPI_SWIGLU;
    constexpr int cols = sw ? 32 : 64;
    const dim3 one((a.N + 31) / 32, (a.M + 31) / 32), two((a.M + 63) / 64, (a.N + cols - 1) / cols), block(64 * kF32Waves);
    auto rounds = [](const dim3 &g) { return ((long)g.x * g.y + 255) / 256; };
    if (rounds(two) * (sw ? 16 : 31) < rounds(one) * 10) hipLaunchKernelGGL((gemm_f32_kernel<EPI, true>), two, block, 0, s, a);
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, false>), one, block, 0, s, a);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int EPI, int BKS = 64, int STAGES = 2, int BSTAGES = STAGES,
          bool STREAM_B = false>
hipError_t run_bf16(const GemmArgs &a, hipStream_t s) {
    const int mt = (a.M + BM - 1) / BM;
    const int cols = EPI == EPI_SWIGLU ? BN / 2 : BN;
    const int nt = (a.N + cols - 1) / cols;
    const int splits =
        (EPI == EPI_ADD_F32 && a.partial && a.splits > 1 && a.K % BKS == 0 && a.K / BKS >= a.splits) ? a.splits : 1;
    if (STREAM_B && mt != 1) return hipErrorInvalidValue;
    if (a.b_blocked && (BKS != 64 || EPI == EPI_SWIGLU || a.K % 64)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, EPI, BKS, STAGES, BSTAGES, STREAM_B>), dim3(mt * nt * splits),
                       dim3(64 * WM * WN), 0, s, a);
    return hipGetLastError();
}

// One 256-row tile per 128 weight rows, the weights streamed once (256x128 tiles of this file): its
// estimated length, measured 1.06 us per K stage and round of 256 workgroups (7B gate/up of 256
// rows 73.8 us), against plan_big's estimate of the same launch.
double stream256_us(int weight_rows, int K) {
    return ((weight_rows + 127) / 128 + 255) / 256 * (K / BK * 1.06 + 6.0);
}

// Split-K projections of 129..256 rows whose 128x128 tiles fill most of the chip with long K runs
// stay on this file's 4-deep rings (7B down, 4 splits: 160 rows 41.9 us against 48.2 on the best
// shape of gemm_big.hip, 256 rows 46.7 against 50.4); shorter runs or fewer workgroups are faster
// there (o 16.2 against 13.7 us, 2048-wide down 22.9 against 17.9 us).
bool ring_split(int M, int N, int K, int splits) {
    const long blocks = (long)((M + 127) / 128) * ((N + 127) / 128) * splits;
    return M > 128 && M <= 256 && blocks >= 192 && K / splits >= 2048;
}

}  // namespace

// Whether gate/up beside another stream's launches (GemmArgs::wide 1, above 256 rows) takes this file's 192x256 tiles
// instead of the light shapes of gemm_big.hip: where their rounds are shorter.  A K stage of a round of 256
// workgroups lasts 1.4 us (7B, 370 rows 93.5 us in one round, 1088 rows 282 in three).  On the 7B shape that is 257 to 384
// rows, for which the light shapes need two rounds of 192x128 tiles, in company 126 to 179 us against 102 to 156 (two
// models, two layers: 320 + 16 rows 755 -> 710 us, 320 + 320 997 -> 935, 64 + 320 783 -> 732), and 641 to 768
// (768 + 128 rows 1183 -> 1164, 768 + 256 1427 -> 1410); over 50 such steps of six shapes 1.6 % on average.
bool gate_up_on_192(int M, int N, int K) {
    const long tiles = (long)((M + 191) / 192) * ((N + 127) / 128);
    return (tiles + 255) / 256 * (K / BK * 1.4 + 4.0) < plan_big(M, N, K, true, 1, true).us;
}

namespace {

// Tile choice per shape, from measurements of the step's projections on MI355X (7B-class layer, cold
// weights unless said otherwise):
//  - M <= 64 (decode-only batches, the LM head): weight streaming; 64x64 tiles (more
//    workgroups) with a 4-deep copy ring keep enough bytes in flight per CU (LM head
//    64 x 32000 x 4096: 70 -> 43 us with warm caches; decode-batch QKV 35 -> 25 us); gate/up
//    on 64x128 tiles (224 workgroups instead of 112: 58.6 -> 43.9 us);
//  - 64 < M <= 128 (decode batches of up to 128 rows): one row tile of 128 rows and a 4-deep
//    ring (128 KiB of LDS), weights streamed: gate/up 66.5 -> 47.3 us, LM head 74.6 -> 66.5 us,
//    down split 4 ways on 128x64 tiles 38.8 -> 32.7 us (M = 96);
//  - 128 < M <= 256: gate/up and stored rows on one 256x128 row tile with the weights streamed once
//    (non-temporal) where that is the shorter estimate, long split-K runs as ring_split says;
//  - everything else above 128 rows that has the chip to itself: gemm_big.hip (370 / 544 / 896
//    rows: gate/up 93.5 / 169.7 / 246.9 -> 84.6 / 129.8 / 190.3 us, down 68.4 / 116.1 / 124.3 ->
//    56.8 / 74.4 / 87.8, o 22.9 / 35.1 / 37.8 -> 18.9 / 25.4 / 33.0; 2048-wide layer, 370 rows:
//    42.5, 26.7, 12.3 -> 31.6, 22.0, 10.3);
//  - beside another stream's launches the large kernel's 256-row tiles leave no registers and no LDS
//    for that stream's small kernels (two models, 1024 + 256 rows, 8 layers: 6.08 against 5.99 ms).
//    Groups of at most 896 rows (GemmArgs::wide 1) take its light shapes (two models, 4 layers, 512 +
//    256 rows 2.58 -> 2.47 ms, 256 + 64 rows 1.43 -> 1.39 against this file's tiles; groups of at most 256
//    rows as above, so on 128 or 144 KB of LDS where this file's tiles are the shorter alone), gate/up on
//    192x256 tiles of this file where their rounds are shorter (gate_up_on_192); beside larger
//    groups (wide 2) this file's tiles stay: split-K projections of 129..256 rows and of more than
//    896 on 256x256 (fewest workgroup-microseconds per flop; the other stream's launches fill the
//    rest; the light shapes take 6.75 instead of 5.99 ms), gate/up above 256 rows on the 192x256,
//    256x256 or 128x128 tiles that need the fewest rounds or pad the rows least.
template <int EPI>
hipError_t dispatch_bf16(const GemmArgs &a, hipStream_t s) {
    const bool big = gemm_big_takes(a) && a.wide < 2;
    if constexpr (EPI == EPI_SWIGLU) {
        if (a.M <= 64) return run_bf16<64, 128, 2, 2, EPI, 64, 4, 4, true>(a, s);
        if (a.M <= 128) return run_bf16<128, 128, 2, 2, EPI, 64, 4, 4, true>(a, s);
        if (big) {
            if (a.wide && a.M > 256 && gate_up_on_192(a.M, a.N, a.K)) return run_bf16<192, 256, 2, 4, EPI>(a, s);
            const BigPlan p = plan_big(a.M, a.N, a.K, true, 1, a.wide);
            // (plan_big's estimate is for weights that several row tiles share; read once, from HBM, they
            // take a fifth longer: 160 / 256 rows of the 7B gate/up est. 57 / 65, measured 64 / 80 us)
            if (a.M > 256 || 1.2 * p.us < stream256_us(2 * a.N, a.K)) return launch_gemm_big(EPI, a, p, s);
        }
        if (a.M <= 256) return run_bf16<256, 128, 4, 2, EPI, 64, 3, 3, true>(a, s);
        if (a.M > 896) {
            // the row tile whose rounds of workgroups over 256 CUs cost least, a round costing
            // its tile's rows
            const long t192 = (long)((a.M + 191) / 192) * ((a.N + 127) / 128);
            const long t256 = (long)((a.M + 255) / 256) * ((a.N + 127) / 128);
            if ((t256 + 255) / 256 * 256 < (t192 + 255) / 256 * 192) return run_bf16<256, 256, 2, 4, EPI>(a, s);
            return run_bf16<192, 256, 2, 4, EPI>(a, s);
        }
        const int pad128 = (a.M + 127) / 128 * 128 - a.M, pad192 = (a.M + 191) / 192 * 192 - a.M;
        const int w128 = (a.M + 127) / 128 * ((a.N + 127) / 128), w192 = (a.M + 191) / 192 * ((a.N + 255) / 256);
        if ((w128 > 512 && w192 <= 256) || pad192 <= pad128) return run_bf16<192, 256, 2, 4, EPI>(a, s);
        return run_bf16<128, 128, 2, 2, EPI>(a, s);
    } else {
        // the blocked LM head of 33..64 rows: 64x128 tiles (16 KB runs per stage) 49.5 -> 46.9 us
        if (EPI == EPI_STORE_F32 && a.b_blocked && a.M > 32 && a.M <= 64)
            return run_bf16<64, 128, 2, 2, EPI, 64, 4, 4, true>(a, s);
        if (a.M <= 64) return run_bf16<64, 64, 2, 2, EPI, 64, 4, 4, true>(a, s);
        const bool split = EPI == EPI_ADD_F32 && a.partial && a.splits > 1;
        if (split && a.M <= 128) return run_bf16<128, 64, 2, 2, EPI, 64, 4, 4, true>(a, s);
        if (EPI != EPI_ADD_F32 && a.M <= 128) return run_bf16<128, 128, 2, 2, EPI, 64, 4, 4, true>(a, s);
        if (a.M <= 128) return run_bf16<128, 128, 4, 2, EPI>(a, s);
        if (big && !(split && ring_split(a.M, a.N, a.K, a.splits))) {
            const BigPlan p = plan_big(a.M, a.N, a.K, false, split ? a.splits : 1, a.wide);
            if (a.M > 256 || EPI == EPI_ADD_F32 || p.us < stream256_us(a.N, a.K)) return launch_gemm_big(EPI, a, p, s);
        }
        // stored rows of 129..256 (the LM head of up to 256 decode rows): one 256-row tile, the
        // weights streamed once
        if (EPI == EPI_STORE_F32 && a.M <= 256) return run_bf16<256, 128, 4, 2, EPI, 64, 3, 3, true>(a, s);
        if (a.wide && ((split && a.M <= 256) || a.M > 896)) return run_bf16<256, 256, 2, 4, EPI>(a, s);
        if (split && a.M <= 256) return run_bf16<128, 128, 2, 2, EPI, 64, 4, 4, false>(a, s);
        return run_bf16<128, 128, 2, 2, EPI>(a, s);
    }
}

}  // namespace

// Split-K factor for a residual-add projection on the bf16 path, matched to the tiles
// dispatch_bf16 uses with it.  Each split takes a run of whole 64-deep stages (the stages dealt
// as evenly as the count allows), at least 512 deep.  1 = no split.
//  - M <= 64 (64x64 tiles): the factor whose workgroups fill the last round over 256 CUs best,
//    the smaller one on a tie;
//  - 64 < M <= 128: 4 (weight streaming wants many workgroups);
//  - M > 128: 4 for the long runs of ring_split, else the factor whose cover of the output
//    (plan_big) and slabs take least time;
//  - M > 896 beside another stream's launches (256x256 tiles, one workgroup per CU): the factor with
//    the least (rounds of workgroups over 256 CUs) x (stages per split), the smaller one on a tie.
int gemm_add_splits(int M, int N, int K, int max_splits, bool wide) {
    auto valid = [&](int s) { return s <= max_splits && K % BK == 0 && K / s >= 512; };
    if (M > 128 && (!wide || M <= 896)) {
        if (valid(4) && ring_split(M, N, K, 4)) return 4;
        return big_splits(M, N, K, max_splits, wide);
    }
    if (M > 896) {
        const int stages = K / BK;
        const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
        int best = 1;
        long best_cost = -1;
        for (int s = 1; s <= max_splits; ++s) {
            if (s > 1 && !valid(s)) continue;
            const long cost = (tiles * s + 255) / 256 * ((stages + s - 1) / s);
            if (best_cost < 0 || cost < best_cost) { best = s; best_cost = cost; }
        }
        return best;
    }
    if (M > 64) {
        int s = 4;
        while (s > 1 && !valid(s)) s /= 2;
        return s;
    }
    const long tiles = (long)((M + 63) / 64) * ((N + 63) / 64);
    auto fill = [](long w) { const long rounds = (w + 255) / 256; return (double)w / (double)(rounds * 256); };
    int best = 1;
    double best_fill = fill(tiles);
    for (int s = 2; s <= max_splits; ++s) {
        if (!valid(s)) continue;
        const double f = fill(tiles * s);
        if (f > best_fill + 1e-9) { best = s; best_fill = f; }
    }
    return best;
}

// Splits (1 or 2) of a QKV projection, whose fp32 rows or partial sums the rotation/append kernel
// reads: two for up to 128 rows (whole-K tiles leave too few workgroups for the weights: 64 rows of
// the 7B shape 42.6 -> 18.6 us, rotation included 25.5), else as the covers' estimates say.  Beside
// another stream's launches one up to 896 rows (the shorter launch is worth less than the partial
// sums' traffic: 256 + 64 rows 1.456 against 1.394 ms) and above 1280, two between.
int gemm_qkv_splits(int M, int N, int K, bool wide) {
    if (K % (2 * BK) || K / 2 < 512) return 1;
    if (M <= 128 || (wide && M > 896 && M <= 1280)) return 2;
    return wide ? 1 : big_splits(M, N, K, 2);
}

// dst [ceil(rows/64)][cols/64][64][64] <- src [rows][cols] (bf16), one 16-byte piece per thread
// step; rows past `rows` in the last row block are zero
__global__ __launch_bounds__(256) void block_weights_kernel(const uint4 *src, uint4 *dst, int rows, int cols) {
    const int cpr = cols / 8;                              // 16-byte pieces per source row
    const size_t total = (size_t)((rows + 63) / 64) * 64 * cpr;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const int c = (int)(i % 8);                        // piece within the block row
        const size_t q = i / 8;
        const int r = (int)(q % 64);                       // row within the block
        const size_t bq = q / 64;                          // block index: rb * (cols / 64) + cb
        const int cb = (int)(bq % (cols / 64));
        const int row = (int)(bq / (cols / 64)) * 64 + r;
        dst[i] = row < rows ? src[(size_t)row * cpr + cb * 8 + c] : uint4{0, 0, 0, 0};
    }
}

hipError_t launch_block_weights(const void *src, void *dst, int rows, int cols, hipStream_t s) {
    const size_t total = (size_t)((rows + 63) / 64) * 64 * (cols / 8);
    const int blocks = (int)std::min<size_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(block_weights_kernel, dim3(blocks), dim3(256), 0, s, (const uint4 *)src, (uint4 *)dst,
                       rows, cols);
    return hipGetLastError();
}

hipError_t launch_gemm(int dtype, int epi, const GemmArgs &a, hipStream_t s) {
    if (a.M <= 0) return hipSuccess;
    if (a.b_blocked && dtype != 1) return hipErrorInvalidValue;
    if (dtype == 1) {
        switch (epi) {
            case EPI_STORE_F32: return dispatch_bf16<EPI_STORE_F32>(a, s);
            case EPI_ADD_F32: return dispatch_bf16<EPI_ADD_F32>(a, s);
            default: return dispatch_bf16<EPI_SWIGLU>(a, s);
        }
    }
    switch (epi) {
        case EPI_STORE_F32: return run_f32<EPI_STORE_F32>(a, s);
        case EPI_ADD_F32: return run_f32<EPI_ADD_F32>(a, s);
        default: return run_f32<EPI_SWIGLU>(a, s);
    }
}

}  // namespace orthrus
