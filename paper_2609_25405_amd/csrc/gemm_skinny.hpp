// Interface of the projections of few rows through small weights (gemm_skinny.hip).
#pragma once

#include "common.hpp"

namespace orthrus {

constexpr int kSkinnyRows = 16, kSkinnyQkvRows = 128;

enum SkinnyEpilogue { SKINNY_STORE = 0, SKINNY_ADD, SKINNY_SWIGLU, SKINNY_QKV };

struct SkinnyArgs {
    const void *A;             // bf16 [M][K], or null: the rows of x through the norm (gain, eps)
    const float *x, *gain;     // fp32 [M][K] residual rows and [K] gain
    float eps;
    const void *B0, *B1;       // weights [N][K]; B1: up rows (SwiGLU)
    int b_blocked;             // B0 in the 64 x 64 blocked layout (SKINNY_STORE only)
    void *out;                 // fp32 [M][N] (store, add) or bf16 [M][N] (SwiGLU)
    int M, N, K, lda, ldo;
    // SKINNY_QKV: N = (nq + 2 nkv) hd; the rows' rotation, q to rope.q_out, k and v into the cache
    // (rope.qkv unused; rope.pos, seq, cs and q_out start at the launch's first row)
    RopeArgs rope;
};
// bf16; M <= kSkinnyRows (SKINNY_QKV: kSkinnyQkvRows), K % 32 == 0
hipError_t launch_skinny(int epilogue, const SkinnyArgs &a, hipStream_t s);
// whether the launch belongs here rather than on the tiled kernels (bf16; weight rows of K each)
bool skinny_takes(int M, int weight_rows, int K);
bool skinny_takes_qkv(int M, int weight_rows, int K);      // the same for SKINNY_QKV
// whether the launch also norms complete rows of x itself
bool skinny_norms(int M, int K);

}  // namespace orthrus
