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
  int xr, pr, pc;                        // set by gemm_skinny.hip's launcher: the tiles of an XCD
  int b_nkc;                             // gemm_skinny.hip: B in fragment order, so many chunks of 32 k (0: rows)
  int frag;                              // gemm_few.hip: both operands in fragment order
  // cell epilogue (cell != 0): N = 128 * ceil(n / 32), column 128 * tile + 32 * gate + unit; bias is [4n] gate-major
  int cell, n;
  const float* h_in; const float* c_in; float* h_out; float* c_out; uint16_t* y; long ldy; float* cs; const int* lens;
  unsigned* status;                      // cleared: nothing in a step waits for another work-group (lstm_sync_status)
};
// gemm_few.hip: C = A B^T for a handful of rows.  The limits lie where it stops being the faster kernel (us here / in gemm_skinny.hip,
// concatenation included).  Cell: a work-group is 4 units of 64 rows, and more than 360 of them (a second round, in part) cost more than the other
// kernel's one: n = 1000, K = 3620 14.6 / 21.2 at 64 rows, 22.3 / 21.3 at 112, 31.7 / 22.7 at 192; n = 704 18.2 / 19.3 at 128, 24.5 / 20.4 at 192; n = 512
// 11.0 / 14.5 at 128, 15.3 / 14.0 at 192; n = 256 10.1 / 12.8 at 192, 15.5 / 13.5 at 240 with K = 2256.  Readout: R = 1000, K = 3620 13.4 / 19.6 at 128 rows, 20.2 / 19.7 at 192.
// Row-major operands: a work-group is 16 columns and takes as long for any K up to 1024, so wide products of more than one row tile leave it: 24 rows,
// N = 8000, K = 512 5.8 / 5.7; 14000 8.8 / 6.3; 20000 10.3 / 8.9, with K = 1000 11.0 / 12.5; 32000 x 1000 23.8 / 18.1; 16 rows, 20000 x 1000 8.7 / 12.4.
constexpr int kFewCellRows = 192, kFewReadoutRows = 192;
inline bool few_cell_pays(long B, long n, long ndir) { return B <= kFewCellRows && (B + 63) / 64 * ((n + 3) / 4) * ndir <= 360; }
inline bool few_rows_pay(long M, long N, long K) { return M <= 16 || (M <= 32 && (N <= 8192 || (K > 896 && N <= 24576))); }
hipError_t launch_few(const SkinnyArgs& a, hipStream_t s);

}  // namespace lstm
