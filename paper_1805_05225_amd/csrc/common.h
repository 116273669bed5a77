// Internal declarations shared by the translation units of the library (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

namespace lstm {

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// round-to-nearest-even float -> bf16 bits, NaN kept quiet
__device__ __forceinline__ uint16_t f2bf_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf_bits2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Storage-type helpers: T is float or bf16_t.
template <typename T> struct Store;
template <> struct Store<float> {
  static constexpr int kBytes = 4;
  static constexpr int kPerChunk = 4;                      // elements in a 16-byte chunk
  __device__ static float load(const void* p, long i) { return ((const float*)p)[i]; }
  __device__ static void store(void* p, long i, float v) { ((float*)p)[i] = v; }
};
template <> struct Store<bf16_t> {
  static constexpr int kBytes = 2;
  static constexpr int kPerChunk = 8;
  __device__ static float load(const void* p, long i) { return bf_bits2f(((const uint16_t*)p)[i]); }
  __device__ static void store(void* p, long i, float v) { ((uint16_t*)p)[i] = f2bf_bits(v); }
};

// K ranges of a product: parts[z][range][m][n] (rows of ldp floats, ldp a multiple of 4; sPz floats per z), added into C (gemm_sum.hip).
struct SumJob {
  const float* parts; void* C; const float* bias;
  int M, N, ksplit, nz;
  long ldp, sPz, ldc, sCz, sbiasz;
  const int* c_rows; const int* m_dev;
  int accumulate, out_bf16;
};
// Sums collected for one launch; `used`: bytes of the parts' memory that they hold until then.
struct SumList {
  static constexpr int kMax = 4;
  int count = 0;
  SumJob j[kMax];
  int first[kMax + 1] = {0, 0, 0, 0, 0};
  size_t used = 0;
  bool add(const SumJob& job);            // false: full
};
hipError_t launch_sums(const SumList& l, hipStream_t s);
// The sum of one product's parts (`bytes` of them): now, or with the others of `later` if that is given and has room.
hipError_t finish_parts(const SumJob& job, size_t bytes, SumList* later, hipStream_t s);

// ------------------------------------------------------------------------------------------
// Hoisted GEMM:  C[m,n] (+)= sum_seg sum_k A(m,k) B(k,n) + bias[n]
//   a_kcontig: A is stored [M][lda] (k contiguous); otherwise [K][lda] (m contiguous).
//   b_kcontig: B is stored [N][ldb] (k contiguous); otherwise [K][ldb] (n contiguous).
// blockIdx.z batches independent problems (pointer strides s*z, in elements).
// nseg > 1 sums over several (A,B) pairs (strides s*seg): used to add both directions' dX.
// lens != NULL masks rows of the K axis: row k is a frame (t = k / Bt, b = k % Bt) and is read
// as zero unless t < lens[b]  (so values stored at padded frames never enter dW_x).
struct GemmArgs {
  const void* A; const void* B; void* C; const float* bias;
  int M, N, K;
  long lda, ldb, ldc;
  long sAz, sBz, sCz, sbiasz;
  int nz;
  int nseg; long sAseg, sBseg;
  int accumulate;            // C += result (float C only)
  const int* lens; int Bt; int T;
  bool a_kcontig, b_kcontig;
  bool in_bf16, out_bf16;
  // Row maps (the fast kernels and the generic one; not the few-rows kernel, and not together with `parts` there):
  const int* a_rows; const int* c_rows;   // k-contiguous A: logical row r of A / C lives at physical row a_rows[r] / c_rows[r]
  int a_phys_rows;                        // rows of A in memory when a_rows is given
  const int* m_dev; const int* k_dev;     // M / K read from device memory (capped by M / K above, which size the grid)
  const int* k_rows; int k_phys_rows;     // both operands k-major: k -> row of A and of B in memory; rows each holds in memory
                                          // (A k-contiguous, B k-major: k_phys_rows > 0 = rows of B, where A's rows are padded up to K)
  float* parts; size_t parts_bytes;       // gemm_tile.hip and gemm_float.hip, which plan their own ranges of K: room for the ranges' parts (their bytes,
                                          // or K stays whole); a second kernel writes C (+)= their sum (`accumulate` honoured)
  SumList* sums;                          // not NULL: that sum is left for the caller's launch_sums
  bool frames;                            // rows of A and C are frames, padded ones included (gemm_float_ranges)
};
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);
// Fast bfloat16 kernel for problems with both operands k-contiguous, rows of whole 8 bytes at 8-byte addresses, K >= 8 and K % 4 == 0
// (launch_gemm routes such problems to it by itself).
bool gemm_nt_ok(const GemmArgs& g);
bool gemm_nn_ok(const GemmArgs& g);                   // (launch_gemm_nt takes these too)
bool gemm_nn_pays(const GemmArgs& g);                 // (the others that are gemm_nn_ok are for launch_gemm_tile)
hipError_t launch_gemm_nt(const GemmArgs& g, hipStream_t s);
// Fast bfloat16 kernel for the opposite storage: both operands k-major (A[K][lda], B[K][ldb], rows of whole 8 bytes),
// float C.  Row k of both operands is row k_rows[k] in memory if k_rows is given (launch_gemm routes to it by itself).
bool gemm_tn_ok(const GemmArgs& g);
hipError_t launch_gemm_tn(const GemmArgs& g, hipStream_t s);
// The same with K in gemm_tn_ranges(g) ranges (1: not worth it, or no room), whose parts go to `parts` and are added as gemm_tile's are.
int gemm_tn_ranges(const GemmArgs& g);
size_t gemm_tn_parts_bytes(long M, long N, long K, int nz);
hipError_t launch_gemm_tn_ranges(const GemmArgs& g, hipStream_t s);
// bfloat16 products with few 256 x 256 tiles, and A k-contiguous x B k-major where gemm_nn_pays does not say otherwise (gemm_tile.hip; launch_gemm routes to it by itself).
// It cuts K into ranges of its own if `parts` holds gemm_tile_parts_bytes.
bool gemm_tile_ok(const GemmArgs& g);
bool gemm_tile_small(long M, long N, int nz);
size_t gemm_tile_parts_bytes(long M, long N, long K, int nz, int nseg);
hipError_t launch_gemm_tile(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_tile_grads(const GemmArgs& dx, const GemmArgs& dwx, const GemmArgs& dwh, hipStream_t s);      // a layer's three gradient products, in one launch
hipError_t launch_gemm_tile_pair(const GemmArgs& g, const GemmArgs& h, hipStream_t s);      // two products of k-major operands, in one launch
// Float storage (gemm_float.hip): operands as they lie in memory, rows 16-byte aligned, K a multiple of 4 for a k-contiguous
// operand; row maps, device-resident M / K and segments as above; K ranges of its own if `parts` holds gemm_float_parts_bytes
// (launch_gemm routes to it by itself; what it does not take goes to the generic kernel).
int gemm_float_ranges(long M, long N, long K, int nz, int nseg, bool frames);      // frames: M counts frames, padded ones included
size_t gemm_float_parts_bytes(long M, long N, long K, int nz, int nseg, bool frames);
bool gemm_float_ok(const GemmArgs& g);
hipError_t launch_gemm_float(const GemmArgs& g, hipStream_t s);
// Products with few rows (gemm_skinny.hip): both operands k-contiguous bfloat16 with 16-byte aligned rows, K % 8 == 0,
// M <= kSkinnyMaxRows, one segment, no row maps, no K ranges: a work-group owns a tile of C, of 32 x 64 to 128 x 128, for the whole K, so bias,
// max(0, .) and the rounding to bfloat16 happen in its epilogue (launch_gemm routes such problems to it by itself).
constexpr int kSkinnyMaxRows = 1024;
bool gemm_skinny_ok(const GemmArgs& g);
hipError_t launch_gemm_skinny(const GemmArgs& g, hipStream_t s);
// the same for rows of any length and alignment (gemm_few.hip)
bool few_any_ok(const GemmArgs& g);
hipError_t launch_few_any(const GemmArgs& g, hipStream_t s);
bool gemm_skinny_pays(long M, long N, int nz);
enum class FewRoute { kHere, kTile, kLarge };          // the kernel for a plain product of few rows: gemm_skinny.hip, gemm_tile.hip, gemm_nt.hip
FewRoute few_rows_route(int M, int N, int K);
// out[B][R] = bf16(max(0, A[B][lda] W^T + bias)): W in the fragment order of launch_pack_rows_both, A's rows at least ceil(K / 32) * 32 columns, zeros past K
hipError_t launch_skinny_readout(const void* A, long lda, const void* Wfrag, const float* bias, void* out, long ldo, int B, int R, int K, hipStream_t s);
// Numbers the frames (t, b) with t < lens[b] in (t, b) order: fidx[number] -> frame, count[0] = how many, count[1] = that rounded up
// to a multiple of 64.
hipError_t launch_frame_map(const int* lens, int T, int B, int* fidx, int* count, hipStream_t s);
// dst[r][0..ld_dst) = src[r][0..C) followed by zeros (16-bit elements)
hipError_t launch_pad_rows(const void* src, void* dst, long R, int C, int ld_dst, hipStream_t s);

// ------------------------------------------------------------------------------------------
// Recurrent part.  Fragment geometry of the 16x16 MFMA used by the step kernels: a 16-byte chunk
// per lane holds kPerChunk consecutive k; lane = g*16 + r with r the row (A) or column (B) inside
// a 16-wide tile and g in 0..3; one chunk index kc covers KC = 4*kPerChunk values of k:
//   k = kc*KC + g*kPerChunk + e.
struct FwdDir {
  const uint4* Wf;    // packed W_h: [unit tile of 8][2 column tiles][nkc][64] chunks
  const uint4* hin;   // h entering the step, fragment order: [row tile of 16][nkc][64] chunks
  void* hout;         // h leaving the step, same layout
  float* gates;       // frame slab [B][4n]: in = x W_x + b, out = activations i|f|g|o
  float* hstate;      // [B][n] float running state
  float* cstate;
  void* y; long ldy;  // row b of this frame's output at y + b*ldy (storage type)
  float* cs;          // frame slab [B][n] or NULL
  void* hprev; long ldh;   // frame slab [B][ldh >= n] (storage type) or NULL
  int t;              // frame index of this step
};
struct FwdArgs {
  FwdDir d[2];
  const int* lens;
  int B, n, nkc, T, ndir, write_gates;
};
hipError_t launch_step_fwd(const FwdArgs& a, bool bf16, hipStream_t s);

struct BwdDir {
  const uint4* Wb;    // packed W_h^T: [unit tile of 16][nkc][64] chunks, k runs over the 4n gate columns
  const uint4* dzin;  // dz of the previous backward step, fragment order [row tile][nkc][64]
  void* dzout;
  const float* gates; // frame slab [B][4n] activations
  const float* cs;    // frame slab [B][n]: cell state after this frame
  const float* cprev; // [B][n]: cell state entering this frame (slab of the neighbouring frame or c0); NULL = 0
  const void* dy; long lddy;
  void* DZ;           // frame slab [B][4n] (storage type)
  float* Dh; float* Dc;   // [B][n] carried gradients
  int t;              // frame of this step (pointwise part)
  int t_next;         // frame whose dz sits in dzin (matmul part)
};
struct BwdArgs {
  BwdDir d[2];
  const int* lens;
  int B, n, nkc, T, ndir, do_matmul, do_pointwise;
};
hipError_t launch_step_bwd(const BwdArgs& a, bool bf16, hipStream_t s);

// Single-launch ("persistent") variants for bfloat16 storage: one launch runs every time step with
// W_h resident in registers.  What crosses work-groups (h_t forward, partial sums of Dh backward)
// travels through a two-slot ring in global memory whose every 8-byte unit carries its values AND a tag
// of the step that wrote it, so a consumer needs no barrier and no fence: it re-reads the ring until every
// tag shows the step it waits for.
//   Forward (h): the K axis of the ring is the unit index; an 8-byte unit carries four consecutive values of one row.
//   |h| <= 1, so bit 14 of a bf16 h (the top bit of the exponent) is always 0; in the fourth value that bit IS the
//   tag - one bit is enough to tell a slot's new contents from what the step two earlier left there - and the reader
//   clears it.  Chunks of 8 values x 64 lanes form MFMA A-fragments exactly as in the per-step kernels.
//   Backward (partial sums of Dh): same unit and tag; the layout is described at the kernels.
// sync[0] is an error word set when a bounded wait expires.
constexpr int kLLValsFwd = 16, kLLSlotsFwd = 16;     // 16 h values  -> 4 units  -> 2 chunks per producer and row
constexpr int kLLMaxNkcFwd = 32;                     // register budget of the kernels (n <= 1024)
constexpr unsigned kLLFwdTagBit = 0x40000000u;       // in the upper dword of a unit: bit 14 of the fourth value
inline int ll_nkc(int n, int slots) { return (int)((((long)(n + 15) / 16) * slots + 31) / 32); }
// packed W_h of one direction; `paired`: in whole tiles of 32 units, for the 8-row kernel
inline size_t ll_wf_bytes(int n, int nkc) { return (size_t)(2 * ((n + 31) / 32)) * 4 * nkc * 1024; }
// The tag bit of the data that step tau consumes (written by step tau - 1 into slot tau & 1; the initial contents of
// slot 0 carry it for tau = 0): it alternates between consecutive uses of a slot and is 1 at a slot's first use, so a
// zero-filled slot never looks written.
__host__ __device__ inline unsigned ll_fwd_tag(unsigned tau) { return ((tau >> 1) & 1u) ^ 1u; }

// How a launch of the bfloat16 kernels maps its work-groups (set by the launcher, explained at wg_coord): unit tiles, row groups
// (of 8 or 16 rows) in the launch, groups per XCD.
struct GridMap { int ntile, nrow, gpx; };

// Rows of different lengths one behind the other in a launch's row places (persistent.hip): built by the set-up launch, read by the loop.
struct PackRows {
  const int* lens; int T, B, slots, tab_steps, max_steps; // slots = 0: not used; more than max_steps steps: steps[0] = -1 and no table
  unsigned* up; unsigned* down; int* steps;               // [group of 8 places][tab_steps][8] frames ascending / descending in time; steps of a group
};
int persist_pack_slots(int T, int B, int n, int ndir, bool backward);
int pack_tab_steps(int T, int B, int slots);
int pack_max_steps(int T, bool backward);
constexpr int kPackMaxSlots = 128, kPackMaxRows = 256;
// y = 0 and the carried cell state at padded frames (which such a launch leaves out; nothing if steps[0] < 0); y [T][B][ndir * n] bfloat16, n even
hipError_t launch_fill_padded(const int* lens, const int* steps, int T, int B, int n, int ndir, void* y, float* const* cs, const float* const* c0, const int* rev, hipStream_t s);

struct PFwdDir {
  const unsigned* tab;  // rows one behind the other: frames in this direction's order
  const uint4* Wf;    // as launch_prep_fwd_ll writes it, or W_h as it lies in memory (w_rows)
  const uint4* Wzero; // one chunk (64 x 16 bytes) of zeros
  uint4* ring0; uint4* ring1;   // [row tile][nkc][64] chunks each
  float* gates;       // [T][B][4n]
  const float* h0; const float* c0; float* hT; float* cT;   // [B][n] each or NULL (zeros; not wanted)
  void* y; long ldy;  // y + column offset of this direction; frame stride B*ldy
  float* cs;          // [T][B][n] or NULL
  void* hprev; long ldh;   // [T][B][ldh >= n] or NULL
  int rev;            // 0: t = tau, 1: t = T-1-tau
};
struct PFwdArgs {
  PFwdDir d[2];
  const int* lens;
  int slots, tab_steps; const int* steps;                 // PackRows (slots = 0: every row has a place of its own)
  int B, n, nkc, T, ndir, write_gates;
  unsigned* sync; unsigned spin_limit;
  unsigned* xcc;      // NULL or one zeroed word per work-group (see PBwdArgs)
  int rt0;            // set by the launcher: first 16-row tile of the batch that this launch handles
  int slab0, slab_tiles;   // likewise (float kernels): first slab of this launch, row tiles per slab
  GridMap map;
  bool plain_launch;  // ordinary instead of cooperative launch (the caller vouches that the device is otherwise idle)
  bool w_rows;        // (persist_fwd_w_rows)
};
hipError_t launch_persist_fwd(const PFwdArgs& a, hipStream_t s);
int persist_fwd_rows(int B, int n, int ndir); // rows per work-group, 8 or 16, which decides how W_h is packed (8: `paired`)
bool persist_fwd_w_rows(int B, int n, int ndir);   // with those 8: does it read W_h as it lies in memory?
int persist_bwd_rows(int B, int n, int ndir);
bool persist_fwd_fits(const PFwdArgs& a);     // would launch_persist_fwd launch anything on this device?
// Float storage (an initial hidden state goes into the pre-activations, as for bfloat16): Wf is the per-step kernel's packed W_h, ring0 / ring1 its
// fragment-ordered h buffers (all by launch_prep_fwd_f32), y / hprev float; nkc = chunks of 16 k.
hipError_t launch_persist_fwd_f32(const PFwdArgs& a, hipStream_t s);
bool persist_fwd_f32_fits(const PFwdArgs& a);
bool persist_f32_pays(int T, int B, int n, int ndir, bool lens, bool plain_launch, bool backward);      // are the float loops faster than the per-step kernels?

struct PBwdDir {
  const unsigned* tab;  // as in PFwdDir, in the order of the backward steps
  const uint4* Wb;    // as launch_prep_bwd_ll writes it
  uint4* ring0; uint4* ring1;
  uint4* wide;        // float storage: scratch as large as a ring
  const float* gates; const float* cs; const float* c0;
  const void* dy; long lddy;
  void* DZ;           // [T][B][4n]
  const float* dhT; const float* dcT; float* dh0; float* dc0;   // [B][n] each or NULL (zeros; not wanted)
  float* dbpart;      // NULL or [2 * row tiles][4n]: slice g receives the bias gradient summed over row group g (8 rows)
  int rev;
};
struct PBwdArgs {
  PBwdDir d[2];
  const int* lens;
  int slots, tab_steps; const int* steps;
  int B, n, T, ndir;
  unsigned* sync; unsigned spin_limit;
  unsigned* xcc;      // NULL or one zeroed word per work-group: lets an exchange group find out whether it shares an XCD
  int rt0;            // set by the launcher: first 16-row tile of the batch that this launch handles
  int slab0, slab_tiles;   // likewise (float kernels): first slab of this launch, row tiles per slab
  GridMap map;
  bool plain_launch;  // ordinary instead of cooperative launch (the caller vouches that the device is otherwise idle)
};
// Does the single-launch backward kernel (partial sums of Dh exchanged; W_h via launch_prep_bwd_ll, ring of
// bwdp_ring_bytes per direction and slot) fit the device for this problem?
bool persist_bwd_fits(const PBwdArgs& a);
hipError_t launch_persist_bwd(const PBwdArgs& a, hipStream_t s);
// Float storage: the same exchange of partial sums in float.  W_h^T via launch_prep_bwd_f32 (bwd_f32_wh_bytes per
// direction), rings of bwd_f32_ring_bytes per direction and slot, zero-filled; gates, cs, dy, DZ float.
bool persist_bwd_f32_fits(const PBwdArgs& a);
hipError_t launch_persist_bwd_f32(const PBwdArgs& a, hipStream_t s);
inline int bwd_f32_nct(int n) { return n <= 256 ? 4 : (n + 127) / 128 * 2; }      // output column tiles (of 16) per wavefront
inline size_t bwd_f32_wh_bytes(int n) { return (size_t)((n + 15) / 16) * 4 * bwd_f32_nct(n) * 16 * 64 * 4; }
inline size_t bwd_f32_ring_bytes(int B, int n) {
  const size_t tiles = (size_t)((n + 15) / 16), rts = 2 * (size_t)(((B > 0 ? B : 1) + 31) / 32);
  return rts * tiles * tiles * 1024;
}
// output column tiles (of 16) per wavefront of the bfloat16 backward kernel: four wavefronts cover n
inline int bwdp_nct(int n) { return n <= 256 ? 4 : n <= 512 ? 8 : 16; }
inline int bwdp8_nct(int n) { return n <= 512 ? bwdp_nct(n) : n <= 640 ? 10 : n <= 768 ? 12 : 16; }      // its 8-row form where every row has a place of its own
inline size_t bwdp_wh_bytes(int n, int nct) { return (size_t)((n + 31) / 32) * 16384 * nct; }           // per direction
inline size_t bwdp_ring_bytes(int B, int n) {                                                      // per direction and slot
  const size_t groups = 2 * (size_t)(((B > 0 ? B : 1) + 15) / 16), tiles = (size_t)((n + 31) / 32);
  return groups * tiles * tiles * 512;
}
// (launch_prep_fwd_ll: W_h in ring order; ring slot 0 = zeros carrying the tag of step 0, ring slot 1 cleared.  The initial state does
// not travel through the ring: its product with W_h is added to the pre-activations of every row's first frame instead, over operands from here.)
// Wide layers, bfloat16 (loop_block.hip): 1024 < n <= 2048, W_h in blocks over the device; one direction per launch.  h0 / c0 / hT / cT / cs / hprev,
// dhT / dcT / dh0 / dc0 may be NULL.  ring: loop_block_ring_bytes (_bwd) bytes; xcc: a word per block; both cleared by the launch, as is *sync.
struct BlockFwdArgs {
  const void* W;                          // launch_pack_blocks
  float* gates;                           // [T][B][4n]
  const float* h0; const float* c0; float* hT; float* cT;
  void* y; long ldy; float* cs; void* hprev; long ldh;
  int rev;
  const int* lens;
  int B, n, T, write_gates;
  char* ring; size_t ring_bytes;
  unsigned* sync; unsigned* xcc; unsigned spin_limit;
  bool plain_launch, first;               // first: of the call's launches; clears the error word
  int row0, ni;                           // set by the launcher: first row; K ranges
};
struct BlockBwdArgs {
  const void* W;                          // W_h as it lies in memory
  const float* gates; const float* cs; const float* c0; const float* dhT; const float* dcT; float* dh0; float* dc0;
  const void* dy; long lddy; void* DZ;
  float* dbpart;                          // [4 ceil(B / 16)][4n] or NULL
  int rev;
  const int* lens;
  int B, n, T;
  char* ring; size_t ring_bytes;
  unsigned* sync; unsigned* xcc; unsigned spin_limit;
  bool plain_launch, first;
  int row0;
};
bool loop_block_width(int n);
bool loop_block_fits(int B, int n, long ld_out);
bool loop_block_pays(int T, int B, int n, int ndir, bool plain_launch, bool backward);      // is it faster than the per-step kernels?      // does the current device hold the launch?
size_t loop_block_ring_bytes(int n);
size_t loop_block_ring_bytes_bwd(int n);
size_t loop_block_wh_bytes(int n);
hipError_t launch_pack_blocks(const void* W_h, const BlockFwdArgs& a, hipStream_t s);      // into a.W; clears what launch_block_fwd of the same arguments wants cleared
hipError_t launch_block_fwd(const BlockFwdArgs& a, hipStream_t s);
hipError_t launch_block_bwd(const BlockBwdArgs& a, hipStream_t s);
int device_capacity(const void* kernel);  // work-groups of 256 threads that the device holds at once, one per compute unit at most

// Narrow layers, all of W_h on one compute unit (loop_small.hip): W_h as it lies in memory, states straight from and to the caller's arrays.
struct SmallFwdDir {
  const void* W; float* gates; const float* h0; const float* c0; float* hT; float* cT;     // h0, c0 [B][n] or NULL (zeros); hT, cT or NULL
  void* y; long ldy; float* cs; void* hprev; long ldh;                                    // as in PFwdDir
  int rev;
};
struct SmallFwdArgs {
  SmallFwdDir d[2];
  const int* lens;
  int B, n, T, ndir, write_gates;
  unsigned* sync;                         // cleared
};
struct SmallBwdDir {
  const void* W; const float* gates; const float* cs; const float* c0; const void* dy; long lddy; void* DZ;
  const float* dhT; const float* dcT; float* dh0; float* dc0;                             // each [B][n] or NULL
  float* db; float* dbpart;               // [4n] or NULL; [ceil(B / 4)][4n], a slice per work-group (B <= 4: straight into db)
  int rev;
};
struct SmallBwdArgs {
  SmallBwdDir d[2];
  const int* lens;
  int B, n, T, ndir, accumulate;
  unsigned* sync;                         // cleared
  unsigned* counters; int ncounters;      // cleared for the products behind the loop
};
bool loop_small_ok(int n);
hipError_t launch_small_fwd(const SmallFwdArgs& a, bool bf16, hipStream_t s);
hipError_t launch_small_bwd(const SmallBwdArgs& a, bool bf16, hipStream_t s);

// A few small products in one launch (gemm_tiny.hip), float or bfloat16 operands in either layout each, any alignment.
struct TinyProduct {
  const void* A; const void* B; void* C; const float* bias;
  int M, N, K;
  long lda, ldb, ldc, sAz, sBz, sCz, sbiasz; int nz;
  int nseg; long sAseg, sBseg;            // sums over segments of K each
  int a_kcontig, b_kcontig, out_bf16, accumulate;
  const int* lens; int Bt, T;             // lens != NULL: k is frame (k / Bt, k % Bt) and A is read as zero unless it is a real one
  int ksplit, tile0;                      // set by the launcher
};
struct TinyGroup { TinyProduct p[3]; int count; };
// Above these multiply-adds the kernels with tiles in LDS are faster.  Measured: Zx of n_in = n = 64, 2560 frames (84 M) 36 / 34 us, of 128 and 2560
// (336 M) 57 / 50; the three products of a backward pass, bfloat16, 1.0 G 124 / 135 us with the loop, 2.0 G 194 / 195, 4.0 G 178 / 155.
constexpr long kTinyZxMacs = 1L << 28, kTinyBwdMacs = 1L << 31;
long tiny_macs(const TinyProduct& p);
// counters: zeroed, tiny_counters() of them; parts: scratch of tiny_parts_bytes()
int tiny_counters(const TinyGroup& g);
size_t tiny_parts_bytes(const TinyGroup& g);
hipError_t launch_gemm_tiny(const TinyGroup& g, bool in_bf16, unsigned* counters, float* parts, hipStream_t s);

// Weight / state packing and small helpers (all enqueue-only).
hipError_t launch_pack_wh_fwd(const void* W_h, uint4* Wf, int n, int nkc, int ndir, bool bf16, hipStream_t s);
hipError_t launch_pack_wh_bwd(const void* W_h, uint4* Wb, int n, int nkc, int ndir, bool bf16, hipStream_t s);
// h (float [ndir][B][n]) -> fragment order, zero padded, written to both ping-pong buffers
hipError_t launch_pack_state(const float* h, uint4* frag0, uint4* frag1, int B, int n, int nkc, int nrt, int ndir,
                             bool bf16, hipStream_t s);
int device_ok();   // 0 if the current device is gfx950, else a negative lstm_status (cached after the first call)
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);                 // p 4-byte aligned, bytes % 2 == 0
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);   // bytes % 4 == 0
// Up to kMax regions cleared by one launch (the set-up of a layer clears half a dozen small buffers; one launch each
// costs more in launch gaps than in work).  Every region 4-byte aligned, bytes % 4 == 0.
struct ZeroRegions {
  static constexpr int kMax = 8;
  void* ptr[kMax];
  size_t words[kMax];
  int first_block[kMax + 1];
  int count;
  bool overflow;
  ZeroRegions() : ptr{}, words{}, first_block{}, count(0), overflow(false) {}
  void add(void* p, size_t bytes);
};
hipError_t launch_fill_zero_many(const ZeroRegions& r, hipStream_t s);
// The set-up of a bfloat16 single-launch loop in one launch: the fills of `z`, W_h in the kernel's order (or fetched), (forward) the initial
// ring, and the frame map of launch_frame_map if fm.fidx is not NULL.
// Copies that ride in a set-up launch (each took a launch of its own, 5 us, most of it the gap): x in padded rows, as launch_pad_rows (x NULL: none), and the initial state as the left operand of
// its product with W_h (h0 NULL: none): out[dir][b][0..ld) = h0[dir][b][0..n) rounded to the storage type, as the recurrence would feed it, then zeros; row[dir][b] = t0 * B + b,
// t0 the row's first frame (reverse: len - 1; a row without frames: one that nobody reads).
struct SetUpCopies {
  const void* x; void* xpad; long x_rows; int x_cols, x_ld;
  const float* h0; void* out; int* row; int ld, rev0, rev1;
  const int* lens; int T, B, n, ndir;
};
struct FrameMapArgs { const int* lens; int T, B; int* fidx; int* count; };
hipError_t launch_prep_fwd_ll(const ZeroRegions& z, const void* W, uint4* Wf, int n, int nkc, int ndir, bool paired, uint4* ring0, uint4* ring1,
                              int nrt, const FrameMapArgs& fm, const PackRows& rows, const SetUpCopies& copies, const GemmArgs* zx, hipStream_t s);
// Wf NULL: W_h is not packed but fetched into the last-level cache (the loop reads it as it lies in memory: PFwdArgs::w_rows).
// zx (few_zx_ok; neither a frame map nor PackRows): the input projection of all frames in the same launch.  It pays for what the compute units take: a
// work-group (32 units, 64 frames) walks all of K, so K times the rounds of 256 of them, and a round of its own costs, too.  A layer's forward pass, us, the
// projection with the set-up / in launches of its own (8 rows, two directions unless said): n = 1000, n_in = 40, 320 frames (5 rounds) 89 / 90, 384 (6) 100 / 100,
// 512 (8) 122 / 118; n = 1024, n_in = 128, 384 frames 105 / 102, 512 127 / 121; n = 1000, n_in = 1000, 256 frames (4) 94 / 99; n_in = 2000, 128 frames (2) 75 / 79;
// n = 520, n_in = 1000, 512 frames (5) 129 / 130; n_in = 2000, 192 frames (2) 77 / 80, 256 (3) 95 / 92; n_in = 4000, 64 frames (1) 56 / 60, 128 (2) 82 / 75.
// Rows of x that are not whole 16 bytes would be copied first: n = 1000, n_in = 620, 384 frames (6 rounds) 114 / 120, 512 (8) 142 / 142.
constexpr int kFewZxRows = 512;
constexpr long kFewZxWalk = 5120;
bool few_zx_ok(const GemmArgs& g);
// The same for the float loops (forward: `p` as launch_persist_fwd_f32 takes it).
hipError_t launch_prep_fwd_f32(const ZeroRegions& z, const void* W, void* Wf, const PFwdArgs& p, const FrameMapArgs& fm, const SetUpCopies& copies, hipStream_t s);
hipError_t launch_prep_bwd_f32(const ZeroRegions& z, const void* W, void* Wb, int n, int ndir, const FrameMapArgs& fm, const SetUpCopies& copies, hipStream_t s);
hipError_t launch_prep_bwd_ll(const ZeroRegions& z, const void* W, uint4* Wb, int n, int ndir, bool paired, int nct, const FrameMapArgs& fm, const PackRows& rows, const SetUpCopies& copies, hipStream_t s);
// db[c] (+)= sum_rows DZ[row][c]; part = float scratch [nsplit][ncols] per direction
// db[dir][c] (+)= sum over the first nslices slices of part[dir][kColsumSlices][ncols]
constexpr int kColsumSlices = 64;
hipError_t launch_colsum(const void* DZ, float* db, float* part, int rows, int ncols, int ndir, long sDZ,
                         bool bf16, int accumulate, hipStream_t s);

// One time step for all rows as a single product (inference, bfloat16 storage; see single_step.hip):
// Wcat[ndir][4n][Kc] = [W_x^T | 0 up to n_in_pad | W_h^T | 0 up to Kc]
hipError_t launch_pack_wcat(const void* W_x, const void* W_h, void* Wcat, int n_in, int n_in_pad, int n, int Kc, int ndir, hipStream_t s);
// Acat[ndir][B][Kc] = [x | 0 | bf16(h[dir]) | 0] in the same column layout (h == NULL: zeros)
// max-pooling in time (time_pool.hip); arg [T'][B][F] bytes, lens_out [B] may be NULL
hipError_t launch_time_pool_fwd(bool bf16, const void* y, long ldy, const int* lens, void* out, long ldo, uint8_t* arg, int* lens_out, int T,
                                int B, int F, int pool, hipStream_t s);
hipError_t launch_time_pool_bwd(bool bf16, const void* dout, long ldo, const uint8_t* arg, const int* lens, void* dy, long ldy, int T, int B,
                                int F, int pool, hipStream_t s);
hipError_t launch_concat_xh(const void* x, const float* h, void* Acat, int B, int n_in, int n_in_pad, int n, int Kc, int ndir, hipStream_t s);
// The same step with the cell update in the product's epilogue (gemm_skinny.hip):
// Wcell[ndir][128 * ceil(n/32)][Kc]: row 128 t + 32 q + u = row q n + 32 t + u of Wcat (zeros for units past n), so that
// a tile of 128 columns holds the four gates of 32 units.  Arguments of the step as for launch_cell_step.
inline size_t wcell_rows(int n) { return (size_t)128 * ((n + 31) / 32); }
hipError_t launch_pack_wcell(const void* W_x, const void* W_h, void* Wcell, int n_in, int n_in_pad, int n, int Kc, int ndir, hipStream_t s);
hipError_t launch_step_cell(const void* Acat, const void* Wcell, const float* bias, const float* h_in, const float* c_in, float* h_out,
                            float* c_out, void* y, long ldy, float* cs, const int* lens, unsigned* status, int B, int n, int Kc, int ndir, hipStream_t s);
// The same step for a handful of rows (gemm_few.hip, few_cell_pays): weights packed in MFMA fragment order (at most wcell_rows(n) x Kc
// elements per direction), K = n_in_pad + n; A is scratch for the concatenated rows in the same order.
hipError_t launch_pack_cell_frag(const void* W_x, const void* W_h, void* out, int n_in, int n_in_pad, int n, int K, int ndir, hipStream_t s);
hipError_t launch_few_cell(const void* x, const float* h_in, void* A, const void* Wfrag, const float* bias, const float* c_in, float* h_out,
                           float* c_out, void* y, long ldy, float* cs, const int* lens, unsigned* status, int B, int n_in, int n_in_pad, int n, int ndir, hipStream_t s);
// out[B][R] = bf16(max(0, [x0 | x1 | x2] W^T + bias)), W in the fragment order of launch_pack_rows_both, A scratch of frag_bytes(B, K)
hipError_t launch_pack_rows_both(const void* W, void* rows, void* frag, int R, int K, int Kp, hipStream_t s);
hipError_t launch_few_readout(const void* x0, long ld0, int k0, const void* x1, long ld1, int k1, const void* x2, long ld2, int k2, void* A,
                              const void* Wfrag, const float* bias, void* out, long ldo, int B, int R, hipStream_t s);
inline size_t frag_bytes(long rows, long K) { return (size_t)((rows + 15) / 16) * ((K + 31) / 32) * 1024; }
// cell update from the pre-activations z = bias + sum of `nparts` partial products, laid out [ndir][nparts][part floats]
// with [B][4n] inside a part.  h_in, c_in [ndir][B][n]: state entering the step (NULL = zeros); h_out, c_out: state
// leaving it (NULL = not wanted); y[B][ldy] (direction d at column d*n); cs[ndir][B][n] or NULL; rows with lens[b] < 1
// keep their state and output zero
hipError_t launch_cell_step(const float* z, long part, int nparts, const float* bias, const float* h_in, const float* c_in, float* h_out,
                            float* c_out, void* y, long ldy, float* cs, const int* lens, unsigned* status, int B, int n, int ndir, hipStream_t s);

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// Do two arrays of `rows` rows share a byte?  Row strides and widths in bytes; column blocks of one matrix (same stride) do not.
inline bool rows_overlap(const void* a, long ld_a, long width_a, const void* b, long ld_b, long width_b, long rows) {
  if (!a || !b || rows < 1 || width_a < 1 || width_b < 1) return false;
  const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  if (a0 + (rows - 1) * ld_a + width_a <= b0 || b0 + (rows - 1) * ld_b + width_b <= a0) return false;
  if (ld_a != ld_b || rows == 1) return true;
  const long d = ((long)(b0 - a0) % ld_a + ld_a) % ld_a;             // column of a's rows in which b's begin
  return d < width_a || d + width_b > ld_a;
}
inline bool bytes_overlap(const void* a, size_t na, const void* b, size_t nb) { return rows_overlap(a, 0, (long)na, b, 0, (long)nb, 1); }

// Host-side set-up that HIP keeps per device (function attributes, what a device is and holds): done once on every
// device the library is used on, whichever thread gets there first.  `done` holds one bit per device ordinal (ordinals
// 64 apart share a bit: the set-up is then simply repeated); the set-up must be idempotent, since two threads may both run it.
template <typename F>
hipError_t once_per_device(std::atomic<unsigned long long>& done, F&& setup) {
  int dev = 0;
  const hipError_t eg = hipGetDevice(&dev);
  if (eg != hipSuccess) return eg;
  const unsigned long long bit = 1ull << (dev & 63);
  if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  const hipError_t e = setup();
  if (e == hipSuccess && dev < 64) done.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace lstm
