// Arguments shared by the two kernels for products with few rows (gemm_skinny.hip, gemm_few.hip).
#pragma once
#include "common.h"

namespace lstm {

struct SkinnyArgs {
  const char* A; const char* B; void* C; const float* bias;
  int M, N, K;
  long lda, ldb, ldc;                    // elements
  long sAz, sBz, sCz, sbiasz; int nz;    // blockIdx.z batches independent problems (the two directions)
  int out_bf16, relu;
  int frag;                              // gemm_few.hip: both operands in fragment order
  // cell epilogue (cell != 0): N = 128 * ceil(n / 32), column 128 * tile + 32 * gate + unit; bias is [4n] gate-major
  int cell, n;
  const float* h_in; const float* c_in; float* h_out; float* c_out; uint16_t* y; long ldy; float* cs; const int* lens;
};
// gemm_few.hip: C = A B^T for a handful of rows.  The limits lie where it stops being the faster kernel (n_in = 2620, n = 1000, us
// here / there, concatenation included): cell 10 / 34 at 12 rows, 23 / 40 at 128, 31 / 40 at 192, 40 / 41 at 256; readout 10 / 20
// at 12, 19 / 21 at 100; row-major operands, N = 20000, 7 / 16 at 12, 11 / 16 at 24, 17 / 17 at 48.
constexpr int kFewRows = 32, kFewCellRows = 192, kFewReadoutRows = 192;
hipError_t launch_few(const SkinnyArgs& a, hipStream_t s);

}  // namespace lstm
