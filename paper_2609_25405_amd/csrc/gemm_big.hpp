// Interface of the large bf16 projections (gemm_big.hip).
#pragma once

#include "common.hpp"

namespace orthrus {

// How a launch covers its output: 256 x 256 tiles on m_main x n_main of it and m_alt x n_alt tiles
// of a second shape from (row_alt, col_alt) on; columns count outputs.
struct BigPlan {
    // second shape: 0 none, 1 128 x 256, 11 64 x 256 (last rows), 2 256 x 192, 3 256 x 128 (last
    // columns); 4 to 10: the second shape covers everything (see launch_shape)
    int shape = 0;
    int m_main = 0, n_main = 0, m_alt = 0, n_alt = 0, row_alt = 0, col_alt = 0;
    int splits = 1;
    int add = 0;      // fp32 rows: add into the output (unsplit) instead of storing
    double us = 0;    // estimated length in microseconds
};
// the cover of [M][N] (swiglu: N gate and N up rows of weights) with the least estimated length; light:
// only of shapes that leave a CU's registers and LDS room for another stream's small kernels
BigPlan plan_big(int M, int N, int K, bool swiglu, int splits, bool light = false);
// the split-K factor (at least 512 deep) whose cover and slabs take least time
int big_splits(int M, int N, int K, int max_splits, bool light = false);
// whether the kernel's addressing covers these operands (K % 64 == 0, rows of at most 8 MB)
bool gemm_big_takes(const GemmArgs &a);
// EPI_STORE_F32, EPI_ADD_F32 (with plan.splits > 1: slabs in a.partial) or EPI_SWIGLU
hipError_t launch_gemm_big(int epi, const GemmArgs &a, const BigPlan &p, hipStream_t s);

}  // namespace orthrus
