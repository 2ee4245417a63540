// LoRA shrink x A^T of the embedding rows (the first half of the low-rank update; the second,
// U B^T, runs inside the projection GEMM's epilogue).  The shared-backbone deployment of the
// paper adapts the generator into the embedding model this way (Section 2, parameter sharing).
//
// bf16 path: one workgroup per 16 rows x 16 columns of U (so one adapter), eight waves splitting K
// eight ways on v_mfma_f32_16x16x32_bf16 with operands loaded straight from global memory, eight K
// steps in flight; a block none of whose rows names its adapter writes zeros and ends.  The eight
// partial blocks are summed in LDS in a fixed order (deterministic), scaled, masked to the
// row's adapter and stored as two bf16 arrays, the rounding of each value and its remainder, so
// the expand can use U to about 16 significant bits (a single bf16 U doubles the adapter
// path's rounding error at 7B shapes).  The launch is a chain of load latencies, so workgroups and
// loads in flight count: 512 rows, four adapters of rank 16, 48 us per projection on 16 workgroups
// of 32 x 64 with one step in flight.  fp32 path: one thread per output, plain dot products.
#include "common.hpp"

namespace orthrus {

namespace {

static_assert(kMaxStepAdapters == 4, "pointers are selected from four");
constexpr int kShrinkWaves = 8, kShrinkAhead = 8;

__global__ __launch_bounds__(64 * kShrinkWaves) void lora_shrink_bf16(LoraShrink p) {
    __shared__ float red[kShrinkWaves][16][17];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = blockIdx.x * 16, c0 = blockIdx.y * 16, ldu = p.n * p.r;
    const int j = c0 / p.r, kk = c0 % p.r;                 // ranks are multiples of 16
    const int rr = (threadIdx.x >> 4) & 15, cc = threadIdx.x & 15;
    const size_t o = (size_t)(m0 + rr) * ldu + c0 + cc;
    const bool mine = m0 + (lane & 15) < p.rows && p.row_adapter[min(m0 + (lane & 15), p.rows - 1)] == j;
    if (__ballot(mine) == 0) {
        if (threadIdx.x < 256 && m0 + rr < p.rows) {
            ((bf16 *)p.u)[o] = (bf16)0.f;
            ((bf16 *)p.u_lo)[o] = (bf16)0.f;
        }
        return;
    }
    const int steps = p.K / 32;
    const int s0 = wave * steps / kShrinkWaves, s1 = (wave + 1) * steps / kShrinkWaves;
    const void *a = j == 0 ? p.a[0] : j == 1 ? p.a[1] : j == 2 ? p.a[2] : p.a[3];
    const bf16 *xr = (const bf16 *)p.x + (size_t)min(m0 + (lane & 15), p.rows - 1) * p.ldx + 8 * (lane >> 4);
    const bf16 *ar = (const bf16 *)a + (size_t)(kk + (lane & 15)) * p.K + 8 * (lane >> 4);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; s += kShrinkAhead) {
        bf16x8 xa[kShrinkAhead], aa[kShrinkAhead];
#pragma unroll
        for (int i = 0; i < kShrinkAhead; ++i) {
            if (s + i >= s1) break;
            xa[i] = *(const bf16x8 *)(xr + 32 * (s + i));
            aa[i] = *(const bf16x8 *)(ar + 32 * (s + i));
        }
#pragma unroll
        for (int i = 0; i < kShrinkAhead; ++i) {
            if (s + i >= s1) break;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[i], aa[i], acc, 0, 0, 0);
        }
    }
    // lane holds column lane % 16, rows 4 (lane / 16) + e
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][(lane >> 4) * 4 + e][lane & 15] = acc[e];
    __syncthreads();
    if (threadIdx.x < 256 && m0 + rr < p.rows) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kShrinkWaves; ++w) sum += red[w][rr][cc];
        const float scale = j == 0 ? p.scale[0] : j == 1 ? p.scale[1] : j == 2 ? p.scale[2] : p.scale[3];
        const float v = p.row_adapter[m0 + rr] == j ? sum * scale : 0.f;
        const bf16 hi = (bf16)v;
        ((bf16 *)p.u)[o] = hi;
        ((bf16 *)p.u_lo)[o] = (bf16)(v - to_f32<bf16>(hi));
    }
}

__global__ __launch_bounds__(256) void lora_shrink_f32(LoraShrink p) {
    const int row = blockIdx.x, ldu = p.n * p.r;
    const float *x = (const float *)p.x + (size_t)row * p.ldx;
    const int ra = p.row_adapter[row];
    for (int c = threadIdx.x; c < ldu; c += 256) {
        const int j = c / p.r, kk = c % p.r;
        float v = 0.f;
        if (ra == j) {
            const float *a = (const float *)p.a[j] + (size_t)kk * p.K;
            for (int i = 0; i < p.K; ++i) v = fmaf(x[i], a[i], v);
            v *= p.scale[j];
        }
        ((float *)p.u)[(size_t)row * ldu + c] = v;
    }
}

}  // namespace

hipError_t launch_lora_shrink(int dtype, const LoraShrink &p, hipStream_t s) {
    if (p.rows <= 0 || p.n <= 0) return hipSuccess;
    if (dtype == 1) {
        if (p.K % 128 || p.r % 16) return hipErrorInvalidValue;
        dim3 grid((p.rows + 15) / 16, p.n * p.r / 16);
        hipLaunchKernelGGL(lora_shrink_bf16, grid, dim3(64 * kShrinkWaves), 0, s, p);
    } else {
        hipLaunchKernelGGL(lora_shrink_f32, dim3(p.rows), dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

}  // namespace orthrus
