// Projections of at most 16 rows (QKV: 128) through small weights (bf16; skinny_takes): a few rows of a small model,
// where a launch is a chain of latencies and a step a chain of launches.  Hence no LDS staging and
// no split-K slabs: a workgroup takes 16 weight rows (two sets of 16 where an epilogue needs
// pairs: gate and up, the two halves of a rotation), its eight waves split K, and each wave loads its
// operands straight into registers in the layout of v_mfma_f32_16x16x32_bf16, up to sixteen K
// steps ahead.  The eight partial tiles meet in LDS and are summed in wave order, and the
// epilogues finish the row: residual add, SwiGLU, rotation with the cache append.  The launch may also norm
// complete rows of x itself (skinny_norms), under the first weights' latency.  4 rows of a 512-wide 8-layer model: 8 launches a layer -> 5 and a step 364 -> 227
// us (projections 5.5 to 10.4 us on the tiled kernels, 3.7 to 5.7 here).
//
// Larger weights stay on the tiled kernels, whose copies to LDS move whole 128-byte lines: one row of
// the 7B shape takes 52 us here against 45 for gate/up, 37.8 against 28.7 for o and down.
#include <algorithm>

#include "gemm_common.hpp"
#include "gemm_skinny.hpp"

namespace orthrus {

namespace {

constexpr int kWaves = 8;
constexpr int kNormK = 1024;      // the longest rows normed here

// SETS: weight row sets of 16 per workgroup.  NORM: A is x normed here.
template <int EPI, int SETS, bool NORM>
__global__ __launch_bounds__(64 * kWaves) void skinny_kernel(SkinnyArgs a) {
    // K steps of weights in flight per register set; a normed row, which takes four times the registers of a bf16
    // one, has all its steps in one (K <= kNormK)
    constexpr int kAhead = NORM ? kNormK / (32 * kWaves) : 8, kLoads = NORM ? 1 : 2;
    __shared__ float red[kWaves][SETS][16][17];
    __shared__ float inv_rms[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half_hd = a.rope.hd / 2;
    if constexpr (EPI == SKINNY_QKV) {
        if (blockIdx.y > 0) {               // this workgroup's 16 rows
            const int m0 = blockIdx.y * kSkinnyRows;
            if (NORM) a.x += (size_t)m0 * a.K;
            else a.A = (const char *)a.A + (size_t)m0 * a.lda * 2;
            a.M -= m0;
            a.rope.pos += m0;
            a.rope.seq += m0;
            a.rope.cs += (size_t)m0 * half_hd;
            a.rope.q_out = (bf16 *)a.rope.q_out + (size_t)m0 * a.rope.nq * a.rope.hd;
            a.rope.Te -= m0;
        }
        a.M = min(a.M, kSkinnyRows);
    }
    // first weight row of each set
    int n0[SETS];
    if constexpr (EPI == SKINNY_QKV) {
        const int per_head = half_hd / 16, head = blockIdx.x / per_head, part = blockIdx.x % per_head;
        n0[0] = head * a.rope.hd + part * 16;
        n0[SETS - 1] = n0[0] + half_hd;
    } else if constexpr (EPI == SKINNY_SWIGLU) {
        n0[0] = n0[SETS - 1] = blockIdx.x * 16;
    } else {
#pragma unroll
        for (int f = 0; f < SETS; ++f) n0[f] = (blockIdx.x * SETS + f) * 16;
    }
    // epilogue thread: row om, column on of each set
    const int om = (tid >> 4) & 15, on = tid & 15;
    const bool writes = tid < 256 && om < a.M;
    // the row's cache slot, looked up before the weights so that its loads are long done after them
    int page = -1, pos = 0, pool = 0;
    bool page_ok = false;
    if constexpr (EPI == SKINNY_QKV) {
        if (writes) {
            pos = a.rope.pos[om];
            pool = om < a.rope.Te ? 0 : 1;
            page = (pool ? a.rope.block_table[1] : a.rope.block_table[0])[(size_t)a.rope.seq[om] * (pool ? a.rope.max_blocks[1] : a.rope.max_blocks[0]) +
                                                                         pos / a.rope.page];
            page_ok = page >= 0 && page < (pool ? a.rope.n_pages[1] : a.rope.n_pages[0]);
        }
    }

    const int steps = a.K / 32;
    const int s0 = wave * steps / kWaves, s1 = (wave + 1) * steps / kWaves;
    const char *wp[SETS];
#pragma unroll
    for (int f = 0; f < SETS; ++f) {
        const int row = min(n0[f] + (lane & 15), a.N - 1);
        const char *base = (const char *)(EPI == SKINNY_SWIGLU && f ? a.B1 : a.B0);
        wp[f] = base + (lane >> 4) * 16 +
                (a.b_blocked ? ((size_t)(row / 64) * (a.K / 64) * 64 + row % 64) * 128 : (size_t)row * a.K * 2);
    }
    auto w_at = [&](int f, int s) {
        return wp[f] + (a.b_blocked ? (size_t)(s >> 1) * 8192 + (s & 1) * 64 : (size_t)s * 64);
    };
    bf16x8 w[kLoads][kAhead][SETS];
    auto load_weights = [&](int s, int set) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (s + i >= s1) break;
#pragma unroll
            for (int f = 0; f < SETS; ++f) w[set][i][f] = *(const bf16x8 *)w_at(f, s + i);
        }
    };
    load_weights(s0, 0);

    const int arow = min(lane & 15, a.M - 1);
    float inv = 0.f;
    if constexpr (NORM) {
        for (int m = wave; m < a.M; m += kWaves) {
            const float *xr = a.x + (size_t)m * a.K;
            float ss = 0.f;
            for (int k = 4 * lane; k < a.K; k += 256) {
                const f32x4 v = *(const f32x4 *)(xr + k);
                ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
            }
            ss = wave_sum(ss);
            if (lane == 0) inv_rms[m] = rsqrtf(ss / (float)a.K + a.eps);
        }
        __syncthreads();
        inv = inv_rms[arow];
    }
    const char *ap = (const char *)a.A + (size_t)arow * a.lda * 2 + (lane >> 4) * 16;
    const float *xp = a.x + (size_t)arow * a.K + (lane >> 4) * 8, *gp = a.gain + (lane >> 4) * 8;
    auto load_a = [&](int s) -> bf16x8 {
        if constexpr (NORM) {
            const f32x4 x0 = *(const f32x4 *)(xp + 32 * s), x1 = *(const f32x4 *)(xp + 32 * s + 4);
            const f32x4 g0 = *(const f32x4 *)(gp + 32 * s), g1 = *(const f32x4 *)(gp + 32 * s + 4);
            u32x4 r;
            r[0] = pack_bf16x2(x0[0] * inv * g0[0], x0[1] * inv * g0[1]);
            r[1] = pack_bf16x2(x0[2] * inv * g0[2], x0[3] * inv * g0[3]);
            r[2] = pack_bf16x2(x1[0] * inv * g1[0], x1[1] * inv * g1[1]);
            r[3] = pack_bf16x2(x1[2] * inv * g1[2], x1[3] * inv * g1[3]);
            return __builtin_bit_cast(bf16x8, r);
        } else {
            return *(const bf16x8 *)(ap + 64 * (size_t)s);
        }
    };
    f32x4 acc[SETS];
#pragma unroll
    for (int f = 0; f < SETS; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int s, int set) {
        bf16x8 av[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (s + i >= s1) break;
            av[i] = load_a(s + i);
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (s + i >= s1) break;
#pragma unroll
            for (int f = 0; f < SETS; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[set][i][f], av[i], acc[f], 0, 0, 0);
        }
    };
    if constexpr (NORM) {
        multiply(s0, 0);
    } else {
        for (int s = s0; s < s1; s += 2 * kAhead) {
            load_weights(s + kAhead, 1);
            multiply(s, 0);
            load_weights(s + 2 * kAhead, 0);
            multiply(s + kAhead, 1);
        }
    }
    // lane holds activation row lane % 16, weight rows 4 (lane / 16) + r of each set
#pragma unroll
    for (int f = 0; f < SETS; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][f][lane & 15][(lane >> 4) * 4 + r] = acc[f][r];
    __syncthreads();
    if (!writes) return;
    float v[SETS];
#pragma unroll
    for (int f = 0; f < SETS; ++f) {
        v[f] = red[0][f][om][on];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) v[f] += red[k][f][om][on];
    }
    if constexpr (EPI == SKINNY_SWIGLU) {
        if (n0[0] + on < a.N) ((bf16 *)a.out)[(size_t)om * a.ldo + n0[0] + on] = (bf16)(silu(v[0]) * v[SETS - 1]);
    } else if constexpr (EPI == SKINNY_QKV) {
        const RopeArgs &q = a.rope;
        const int head = n0[0] / q.hd, i = n0[0] % q.hd + on;
        if (!page_ok && head == q.nq && i == 0) flag_error(q.err, ORTHRUS_DEVERR_PAGE);
        if (head < q.nq + q.nkv) {
            const float2 cs = q.cs[(size_t)om * half_hd + i];
            const float y1 = v[0] * cs.x - v[SETS - 1] * cs.y, y2 = v[SETS - 1] * cs.x + v[0] * cs.y;
            if (head >= q.nq && !page_ok) return;
            bf16 *dst = head < q.nq ? (bf16 *)q.q_out + ((size_t)om * q.nq + head) * q.hd
                                    : (bf16 *)(pool ? q.k_cache[1] : q.k_cache[0]) +
                                          (((size_t)page * q.nkv + (head - q.nq)) * q.page + pos % q.page) * q.hd;
            dst[i] = (bf16)y1;
            dst[i + half_hd] = (bf16)y2;
        } else if (page_ok) {
            bf16 *dst = (bf16 *)(pool ? q.v_cache[1] : q.v_cache[0]) +
                        ((size_t)page * q.nkv + (head - q.nq - q.nkv)) * q.hd * q.page + pos % q.page;
            dst[(size_t)i * q.page] = (bf16)v[0];
            dst[(size_t)(i + half_hd) * q.page] = (bf16)v[SETS - 1];
        }
    } else {
#pragma unroll
        for (int f = 0; f < SETS; ++f) {
            if (n0[f] + on >= a.N) continue;
            float *o = (float *)a.out + (size_t)om * a.ldo + n0[f] + on;
            *o = EPI == SKINNY_ADD ? *o + v[f] : v[f];
        }
    }
}

template <int EPI, int SETS>
hipError_t go(const SkinnyArgs &a, int blocks, hipStream_t s) {
    const int row_tiles = (a.M + kSkinnyRows - 1) / kSkinnyRows;
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks, row_tiles), dim3(64 * kWaves), 0, s, a);
        return hipGetLastError();
    };
    if constexpr (EPI == SKINNY_SWIGLU || EPI == SKINNY_QKV) {
        if (!a.A) return run(skinny_kernel<EPI, SETS, true>);
    }
    return run(skinny_kernel<EPI, SETS, false>);
}

}  // namespace

bool skinny_takes(int M, int weight_rows, int K) {
    // at 16 MB one row still gains (2048-wide shape, a step of 1 row 146.8 -> 136.1 us), twelve rows no
    // longer do (178.3 against 182.8 us); at 2 MB all do
    return M <= kSkinnyRows && K % 32 == 0 && (size_t)weight_rows * K * 2 <= (size_t)(M <= 4 ? 16 : 4) << 20;
}

// QKV of 17 to 128 rows, whose rotation and append else are a launch of their own: 16 rows a workgroup, so each row
// tile reads the weights again, from L2.  Worth it while these reads are at most 28 MB: 512-wide, 6 layers, 17 rows 259 ->
// 234 us, 128 rows 371 -> 326; 1024-wide (3 MB) 128 rows 416 -> 394; 2048-wide (4 MB) 64 rows 414 -> 389; two models, 512-wide, 4
// layers, where the host's launches bound the step, 20 + 20 rows 283 -> 253.  At 38 MB equal or 4 to 7 % slower, at
// 75 MB 4 to 9 %.
bool skinny_takes_qkv(int M, int weight_rows, int K) {
    const size_t row_tiles = (M + kSkinnyRows - 1) / kSkinnyRows;
    return skinny_takes(M, weight_rows, K) ||
           (M <= kSkinnyQkvRows && K % 32 == 0 && (size_t)weight_rows * K * 2 * row_tiles <= (size_t)28 << 20);
}

// Every workgroup sums the squares of its rows, two rows a wave with 16 and a load a 256 columns each, and reads them a second
// time as fp32: worth the norm's launch of 4 us while it is short.  Steps of 6 layers, normed here against by a launch:
// 512-wide, 1 / 8 / 16 rows 133 / 148 / 167 us against 149 / 161 / 170; 1024-wide, 1 / 8 / 16 rows 154 / 171 / 200
// against 160 / 172 / 182; 1536-wide, 1 row 179 against 175; 4096-wide, 1 / 16 rows 297 / 428 against 245 / 295.
bool skinny_norms(int M, int K) { return K <= kNormK && std::min(M, kSkinnyRows) * K <= 8192; }

hipError_t launch_skinny(int epilogue, const SkinnyArgs &a, hipStream_t s) {
    if (a.M <= 0) return hipSuccess;
    if (a.M > (epilogue == SKINNY_QKV ? kSkinnyQkvRows : kSkinnyRows) || a.K % 32 || (a.b_blocked && (epilogue != SKINNY_STORE || a.K % 64)) || (!a.A && (a.K > kNormK || (epilogue != SKINNY_SWIGLU && epilogue != SKINNY_QKV))))
        return hipErrorInvalidValue;
    switch (epilogue) {
        case SKINNY_STORE: return go<SKINNY_STORE, 2>(a, (a.N + 31) / 32, s);
        case SKINNY_ADD: return go<SKINNY_ADD, 1>(a, (a.N + 15) / 16, s);
        case SKINNY_SWIGLU: return go<SKINNY_SWIGLU, 2>(a, (a.N + 15) / 16, s);
        case SKINNY_QKV:
            if (a.rope.hd % 32 || a.N != (a.rope.nq + 2 * a.rope.nkv) * a.rope.hd) return hipErrorInvalidValue;
            return go<SKINNY_QKV, 2>(a, a.N / 32, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace orthrus
