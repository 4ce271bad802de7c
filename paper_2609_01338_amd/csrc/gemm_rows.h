// Launcher of the GEMM in tiles of 32 to 128 rows (gemm_rows.hip).
#pragma once
#include "mz_kernels.h"

namespace mzk {

// As gemm_q4.hip's tiles, with row_tile (32, 64 or 128) x 128-column tiles or
// 128 x 256; kEpiPartial: n_split ranges of k_steps K steps of 64, sums to
// y float [split][m][n].
void launch_gemm_rows(const void* x, const int32_t* a_rows, int m, int n, int k, const void* w, int epilogue, void* y,
                      hipStream_t s, int row_tile, int col_tile, int n_split = 1, int k_steps = 0,
                      const GemmRope& ea = GemmRope{});

}  // namespace mzk
