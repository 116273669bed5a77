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
// concatenation included).  Cell: a work-group is 4 units of 64 rows, and the second round of 256, in part, costs as
// much as the other kernel's one.  us of calls in a graph: n = 1000, K = 3620 14.6 / 21.2 at 64 rows, 22.3 / 21.3 at 112, 31.7 / 22.7 at 192; n = 512 11.0 / 14.5 at 128, 15.3 / 14.0 at 192.  Up to 16
// rows (no concatenation) it takes 11.8 whatever K, the other kernel 10.4 for K = 860, 11.2 for 1150, 12.4 for 1460 (792, 816 and 1000 units, both directions), 1.3 to 1.5 times as long from 2000 on;
// 17 to 64 rows are as long here or shorter up to two rounds (384 to 512 work-groups, K from 700 to 2800: 0.76 to 1.12 times the other, 0.96 in the mean).  A third round: 1.1 to 1.4 times.  Readout: R = 1000, K = 3620 13.4 / 19.6 at 128 rows, 20.2 / 19.7 at 192.
// Row-major operands: a work-group is 16 columns and takes as long for any K up to 1024, so wide products of more than one row tile leave it: 24 rows,
// N = 8000, K = 512 5.8 / 5.7; 14000 8.8 / 6.3; 20000 10.3 / 8.9, with K = 1000 11.0 / 12.5; 32000 x 1000 23.8 / 18.1; 16 rows, 20000 x 1000 8.7 / 12.4.
constexpr int kFewCellRows = 192, kFewReadoutRows = 192;
inline bool few_cell_pays(long B, long n, long ndir, long K) {
  const long groups = (B + 63) / 64 * ((n + 3) / 4) * ndir;
  return B <= kFewCellRows && (groups <= 256 || (B <= 16 ? groups <= 512 && K >= 1300 : groups <= (B <= 64 ? 512 : 360)));
}
inline bool few_rows_pay(long M, long N, long K) { return M <= 16 || (M <= 32 && (N <= 8192 || (K > 896 && N <= 24576))); }
hipError_t launch_few(const SkinnyArgs& a, hipStream_t s);

}  // namespace lstm
