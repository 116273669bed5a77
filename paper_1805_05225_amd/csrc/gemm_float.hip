// The hoisted products in float storage (paper Sec. 3: work taken out of the recurrent loop), float in, float out, operands used
// as they lie in memory:
//     <AK, BK> = <true,  false>   Zx   = X W_x + b      A[M][K] rows of frames,  B[K][N]
//                <true,  true >   dX   = DZ W_x^T       A[M][K],                 B[N][K]     (summed over `nseg` directions)
//                <false, false>   dW   = X^T DZ         A[K][M], B[K][N]: a row per frame in both
//     C[z][M][N] (+)= sum_seg sum_k A . B  (+ bias[N])
//
// Tile 128 x 128, four wavefronts of 64 x 64 (4 x 4 MFMA blocks), k advances 32 per stage, two stages in LDS
// (65 KiB: two work-groups per compute unit, so one's barrier and waits hide behind the other's MFMAs).  The operands
// go from global memory straight into LDS (16 bytes per lane, no staging registers, no LDS store instructions); a
// wavefront-load writes 1 KiB, lane l its bytes 16 l .., and what a lane fetches is chosen so that the fragment
// reads meet no bank conflicts:
//   * k-major operand (a memory row is one k): a lane wants eight k-rows of ONE column, column = lane % 16 of a
//     block - 16 lanes reading 16 consecutive floats, no transposition needed.  A
//     stage is 16 pieces of 1 KiB + 16 bytes; piece p holds k-rows p and p + 16 of the stage (512 bytes each).
//   * k-contiguous operand (a memory row is a row of the tile): a stage is 128 rows of 128 bytes, unpadded; the
//     16-byte slot s of row r holds k-chunk s ^ ((r >> 1) & 7).  A lane reads 16 bytes: four consecutive k of its row.
// The eight k of a fragment's lane group q (0..3) are 16 G + 4 q + s, s (0..3), G (0..1): two reads of 16 bytes, or, k-major, eight of 4
// (the four lane groups' pieces lie 4 x 1040 bytes apart, 16 banks from one another).  Both operands follow it, so every k meets its partner.
//
// The matrix cores multiply bfloat16 sixteen times as fast as float, so a float goes as the sum of three bfloat16 (`split`: its 24 bits,
// exactly) and a product as the six of their nine products that matter: 16 x 16 x 32 at 6 x 16 cycles instead of 8 x 32.  The five small ones have
// sums of their own: what the matrix cores cut off where they add to a large sum would otherwise be cut off six times.  Against 64 bits the error is a
// third of the float MFMA's (sum of K products of normal values, root mean square over that of the result: K = 64 0.5e-7 against 1.4e-7, 620
// 1.4e-7 against 4.5e-7, 8000 5.7e-7 against 1.6e-6), for positive values half, and as large where single products dominate the
// sums (lognormal, sigma 3).
// Both operands are multiplied by 2^24 before they are split: the last bit of the smallest float, 2^-149, is then a normal bfloat16 number, so the parts are exact for
// every float below 2^104 in magnitude (as they stand, from 2^-110 up only: 2^-120 times 2^60 came out wrong by 6e-5 of itself).  What is not below that, and
// sums from 2^80 on, end as NaN or infinity; a tile where a result says so is computed again with float MFMAs (16x16x4).  Nothing else depends on the values (small
// results used to: dX of 2400 frames, 620 x 4000, ordinary gradients 188 us, ones that halve 300 times on their way back 448; now 199 and 198).
// Bound by the splitting, 416 vector instructions of 4 cycles for 96 products of 16, which is therefore cut into the products, and by power.
// 4096^3: nn 1060 -> 727 us, nt 1025 -> 702, tn 1080 -> 755 (182 to 196 TFLOP/s, where float MFMAs have a peak of 157);
// 1920 x 8000 x 620 200 -> 121 us.  The factor's 64 instructions are 3 to 7 % of that (694, 655 and 728 without; differences by dot products of two
// bfloat16, which drop the parts' unpacking, 787, 743 and 787).
// The MFMA takes the B fragment (columns n) as its row operand and the A fragment as its column operand: a lane then
// holds four CONSECUTIVE n of one row m of C and stores them as 16 bytes.
// Rows of a k-contiguous A (and of C) may be mapped (`a_rows`, `c_rows`, `m_dev`: the packed list of real frames), as
// may the k-rows of a k-major pair (`k_rows`, `k_dev`), looked up one stage ahead.
#include "common.h"
#include <algorithm>

namespace lstm {
namespace {

constexpr int kTile = 128, kKS = 32;
constexpr int kPiece = 1024 + 16;                // k-major: bytes per piece (k-rows p and p + 16, padding)
constexpr int kOp = 16 * kPiece;                 // one operand, one stage (a k-contiguous one uses 16 KiB of it)
constexpr int kStage = 2 * kOp;
constexpr int kLds = 2 * kStage;                 // 66 560
constexpr int kBufFlags = 0x00020000;            // raw buffer descriptor word 3 for gfx9-family devices
constexpr unsigned kParked = 0x7ffffff0u;        // offset outside every descriptor: the load returns zeros

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

struct FArgs {
  const char* A; const char* B; float* C; const float* bias;
  int M, N, K;
  long lda, ldb, ldc;                            // elements
  long sAz, sBz, sCz, sbiasz;
  int nseg; long sAseg, sBseg;
  int accumulate;
  const int* a_rows; const int* c_rows; int a_phys_rows; const int* m_dev;
  const int* k_rows; int k_phys_rows; const int* k_dev;
  int ksplit;                                    // > 1: K range r stores its part at parts + (z * ksplit + r) * M * ldp, rows packed
  float* parts; long ldp;                        // (of eight ranges, range r is worked on by XCD r alone)
  int tiles_m, tiles_n, per_xcd;
  unsigned a_bytes, b_bytes;                     // extent of one segment of A / B in memory
};

// A buffer load whose data goes to LDS (M0 = wavefront-uniform LDS byte address; lane l writes M0 + 16 l).  Written as
// assembly so that the compiler does not make later LDS reads wait for loads that fill the other stage; the kernel
// orders them with an explicit vmcnt(0) and the barrier of every stage.  Nothing else here uses M0.
__device__ __forceinline__ void load_to_lds_b128(const u32x4& rsrc, unsigned lds_addr, unsigned voff, unsigned soff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ u32x4 make_rsrc(const void* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
  r[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane(bytes);
  r[3] = kBufFlags;
  return r;
}

// A float times 2^24 is the sum of three bfloat16 (8 + 8 + 8 bits, each rounded to nearest, the last exactly); what the six products leave out is below 2^-25 of theirs.
struct Parts { u32x4 p[3]; };
constexpr float kScale = 0x1p24f;
constexpr int kPairA[6] = {0, 0, 1, 1, 0, 2}, kPairB[6] = {0, 1, 0, 1, 2, 0};
__device__ __forceinline__ Parts split(const float (&x)[8]) {
  Parts r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo = x[2 * e] * kScale, hi = x[2 * e + 1] * kScale;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      typedef __attribute__((ext_vector_type(2))) float f32x2;
      typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
      const unsigned v = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
      r.p[p][e] = v;
      lo -= __uint_as_float(v << 16);
      hi -= __uint_as_float(v & 0xffff0000u);
    }
  }
  return r;
}
__device__ __forceinline__ f32x4 mma(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <int N, int V> __device__ __forceinline__ void interleave() {       // N times a product and V vector instructions
#pragma unroll
  for (int e = 0; e < N; ++e) {
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x2, V, 0);
  }
}

template <bool AK, bool BK>
__device__ __forceinline__ void gemm_float_body(const FArgs& g) {
  static_assert(AK || !BK, "a k-major A with a k-contiguous B is not a product of the layer");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // Work-groups are dealt to the eight XCDs round-robin: an XCD takes a run of consecutive tiles, column-major, i.e.
  // all row tiles of a few tile columns - the A panels and those few B panels are what its L2 has to hold.
  // With eight K ranges every XCD takes ALL tiles for one eighth of K instead: its L2 then holds that
  // eighth of B for good and streams that eighth of A once, and no operand byte is fetched by two XCDs.  The tiles
  // of one row panel (same rows of A) are neighbours in launch order, so they run side by side.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const bool to_parts = g.ksplit > 1, by_range = g.ksplit == 8;
  const int t = by_range ? slot : xcd * g.per_xcd + slot;
  if ((!by_range && slot >= g.per_xcd) || t >= g.tiles_m * g.tiles_n) return;
  const int m0 = (by_range ? t / g.tiles_n : t % g.tiles_m) * kTile, n0 = (by_range ? t % g.tiles_n : t / g.tiles_m) * kTile;
  const int M = g.m_dev ? min(g.M, *g.m_dev) : g.M;              // the grid is sized for g.M; surplus tiles leave at once
  if (m0 >= M) return;
  const int ksplit = g.ksplit;
  const int z = by_range ? blockIdx.y : blockIdx.y / ksplit, ks = by_range ? xcd : blockIdx.y - z * ksplit;
  const int K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  const int sps = max((K + kKS - 1) / kKS, 1);                   // stages per segment; what lies past K arrives as zeros
  const int nstage = K > 0 ? sps * g.nseg : 0;
  const int it0 = (int)((long)nstage * ks / ksplit);
  const int total = (int)((long)nstage * (ks + 1) / ksplit) - it0;
  if (total <= 0 && !to_parts && g.accumulate) return;           // nothing to add

  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;
  // ---- loads ----
  // k-major operand: wavefront-load i of this wavefront writes piece p = 4 wave + i; its lower 32 lanes fetch k-row p
  // of the stage, the upper 32 k-row p + 16; lane l fetches columns 4 (l % 32) .. + 3 of the tile.
  const int half = lane >> 5, chunk32 = lane & 31;
  const int k_lane = 16 * half + 4 * wave;                       // k of wavefront-load 0 inside a stage; load i adds i
  const long krows_mem = g.k_phys_rows > 0 ? g.k_phys_rows : K;  // rows that a k-major operand has in memory
  const bool am_col_ok = m0 + chunk32 * 4 < g.M, bm_col_ok = n0 + chunk32 * 4 < g.N;
  const unsigned am_col = (unsigned)(m0 + chunk32 * 4) * 4u, bm_col = (unsigned)(n0 + chunk32 * 4) * 4u;
  // k-contiguous operand: wavefront-load i writes tile rows 32 wave + 8 i .. + 7; lane l fills slot l % 8 of row l / 8
  // of those, i.e. fetches k-chunk (l % 8) ^ ((row >> 1) & 7).  The rows do not change from stage to stage.
  unsigned ak_row[4], bk_row[4];                                 // byte offset of the lane's row (kParked: no such row)
  int ak_kc[4], bk_kc[4];                                        // first k of the chunk the lane fetches, within a stage
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 32 * wave + 8 * i + (lane >> 3);
    const int kc = 4 * ((lane & 7) ^ ((r >> 1) & 7));
    ak_kc[i] = bk_kc[i] = kc;
    ak_row[i] = bk_row[i] = kParked;
    if (AK) {
      long ra = m0 + r;
      const long rows_mem = g.a_rows ? g.a_phys_rows : g.M;
      if (ra < M) {
        if (g.a_rows) ra = g.a_rows[ra];
        if (ra >= 0 && ra < rows_mem) ak_row[i] = (unsigned)(ra * g.lda * 4);
      }
    }
    if (BK) {
      const long rb = n0 + r;
      if (rb < g.N) bk_row[i] = (unsigned)(rb * g.ldb * 4);
    }
  }
  auto lookup = [&](int rel_it) -> int4 {                        // memory rows of the four k this lane fetches (k-major pair)
    const int it = it0 + rel_it, seg = it / sps;
    const int k = (it - seg * sps) * kKS + k_lane;
    if (!AK && !BK && g.k_rows && rel_it < total) return *(const int4*)(g.k_rows + k);   // (readable up to a multiple of 64)
    return make_int4(k, k + 1, k + 2, k + 3);
  };
  auto issue = [&](int rel_it, int buf, const int4& rows) __attribute__((always_inline)) {
    const int it = it0 + rel_it, seg = it / sps;
    const int k0 = (it - seg * sps) * kKS;
    const u32x4 ra = make_rsrc(g.A + (g.sAz * z + g.sAseg * seg) * 4, g.a_bytes);
    const u32x4 rb = make_rsrc(g.B + (g.sBz * z + g.sBseg * seg) * 4, g.b_bytes);
    const int r[4] = {rows.x, rows.y, rows.z, rows.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool row_ok = k0 + k_lane + i < K && r[i] >= 0 && r[i] < krows_mem;
      if (AK) {
        const bool ok = ak_row[i] != kParked && k0 + ak_kc[i] < K;
        load_to_lds_b128(ra, lds_base + buf * kStage + (4 * wave + i) * 1024, ok ? ak_row[i] + (unsigned)ak_kc[i] * 4u : kParked, (unsigned)k0 * 4u);
      } else {
        load_to_lds_b128(ra, lds_base + buf * kStage + (4 * wave + i) * kPiece,
                         row_ok && am_col_ok ? (unsigned)r[i] * (unsigned)(g.lda * 4) + am_col : kParked, 0u);
      }
      if (BK) {
        const bool ok = bk_row[i] != kParked && k0 + bk_kc[i] < K;
        load_to_lds_b128(rb, lds_base + buf * kStage + kOp + (4 * wave + i) * 1024, ok ? bk_row[i] + (unsigned)bk_kc[i] * 4u : kParked, (unsigned)k0 * 4u);
      } else {
        load_to_lds_b128(rb, lds_base + buf * kStage + kOp + (4 * wave + i) * kPiece,
                         row_ok && bm_col_ok ? (unsigned)r[i] * (unsigned)(g.ldb * 4) + bm_col : kParked, 0u);
      }
    }
  };

  // ---- fragment reads ----
  // Lane l = 16 q + i16.  k-major: k-row 16 G + 4 q + s -> piece 4 q + s, half G, column block * 16 + i16.
  // k-contiguous: row block * 16 + i16, k-chunk 4 G + q in slot (4 G + q) ^ ((row >> 1) & 7) (the blocks' row offsets
  // are multiples of 16, so the XOR term depends on i16 only).
  const int q = lane >> 4, i16 = lane & 15;
  const int sw = (i16 >> 1) & 7;
  const char* fa_base[2];                                        // per group G (k-major: the same for both)
  const char* fb_base[2];
#pragma unroll
  for (int G = 0; G < 2; ++G) {
    fa_base[G] = AK ? lds + (wm * 64 + i16) * 128 + (((4 * G + q) ^ sw) * 16) : lds + 4 * q * kPiece + (wm * 64 + i16) * 4 + G * 512;
    fb_base[G] = BK ? lds + kOp + (wn * 64 + i16) * 128 + (((4 * G + q) ^ sw) * 16) : lds + kOp + 4 * q * kPiece + (wn * 64 + i16) * 4 + G * 512;
  }
  f32x4 acc[4][4], low[4][4];                                    // [m block][n block]; element v: n = 4 q + v
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = low[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  int4 rows_next;
  auto stages = [&](auto&& products) __attribute__((always_inline)) {
    rows_next = lookup(0);
    if (total > 0) {
      issue(0, 0, rows_next);
      rows_next = lookup(1);
    }
    for (int it = 0; it < total; ++it) {
      const int cur = it & 1;
      __builtin_amdgcn_s_waitcnt(0x0070);          // vmcnt(0) lgkmcnt(0): this wavefront's loads of stage `it` (and the look-up) are in
      __syncthreads();                             // everybody's are, and everybody has finished reading the other buffer
      if (it + 1 < total) issue(it + 1, cur ^ 1, rows_next);
      rows_next = lookup(it + 2);
      // (fenced: left alone, the compiler moves each read down to its first use and waits for it there)
      __builtin_amdgcn_sched_barrier(0);
      products(cur);
    }
  };
  stages([&](int cur) __attribute__((always_inline)) {
    // the eight k of a lane's fragment: k = 16 G + 4 q + s, element 4 G + s
    auto raw_a = [&](int blk, float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        if (AK) {
          const float4 v = *(const float4*)(fa_base[G] + cur * kStage + blk * 2048);
          x[4 * G] = v.x; x[4 * G + 1] = v.y; x[4 * G + 2] = v.z; x[4 * G + 3] = v.w;
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) x[4 * G + s] = *(const float*)(fa_base[G] + cur * kStage + s * kPiece + blk * 64);
        }
      }
    };
    auto raw_b = [&](int blk, float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int G = 0; G < 2; ++G) {
        if (BK) {
          const float4 v = *(const float4*)(fb_base[G] + cur * kStage + blk * 2048);
          x[4 * G] = v.x; x[4 * G + 1] = v.y; x[4 * G + 2] = v.z; x[4 * G + 3] = v.w;
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) x[4 * G + s] = *(const float*)(fb_base[G] + cur * kStage + s * kPiece + blk * 64);
        }
      }
    };
    // Operands are split two products ahead, between the products: a split is 52 instructions of 4 cycles, six products are 96 cycles.
    Parts a[4], b[2];
    float x[2][8];
    auto pair = [&](int m, int n) __attribute__((always_inline)) {
#pragma unroll
      for (int o = 5; o >= 0; --o) {                       // (the smallest first)
        f32x4& to = o == 0 ? acc[m][n] : low[m][n];
        to = mma(b[n & 1].p[kPairB[o]], a[m].p[kPairA[o]], to);
      }
    };
    raw_a(0, x[0]);
    raw_b(0, x[1]);
    a[0] = split(x[0]);
    raw_a(1, x[0]);
    b[0] = split(x[1]);
    raw_a(2, x[1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      pair(m, 0);
      Parts& to = m < 3 ? a[m + 1] : b[1];
      to = split(x[m & 1]);
      if (m == 0) raw_a(3, x[0]);
      else raw_b(m, x[m & 1]);
      interleave<6, 7>();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int n = 1; n < 4; ++n) {
#pragma unroll
      for (int m = 0; m < 4; ++m) pair(m, n);
      if (n < 3) b[(n + 1) & 1] = split(x[(n + 1) & 1]);
      interleave<24, 2>();
      __builtin_amdgcn_sched_barrier(0);
    }
  });
  bool odd = false;                                              // (see above)
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        acc[m][n][v] += low[m][n][v];
        odd |= !(__builtin_fabsf(acc[m][n][v]) < __builtin_inff());
        acc[m][n][v] *= 1.f / (kScale * kScale);
      }
  if (__builtin_expect(__syncthreads_or(odd), 0)) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[m][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
    stages([&](int cur) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {                        // e = 4 G + s
        const int G = e >> 2, sx = e & 3;
        float fa[4], fb[4];
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
          fa[blk] = *(const float*)(fa_base[G] + cur * kStage + (AK ? sx * 4 + blk * 2048 : sx * kPiece + blk * 64));
          fb[blk] = *(const float*)(fb_base[G] + cur * kStage + (BK ? sx * 4 + blk * 2048 : sx * kPiece + blk * 64));
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int n = 0; n < 4; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[n], fa[m], acc[m][n], 0, 0, 0);
      }
    });
  }

  // Epilogue: lane l holds C[m = block_m * 16 + l % 16][n = block_n * 16 + 4 (l / 16) .. + 3].
  float* C = to_parts ? g.parts + ((long)z * ksplit + ks) * g.M * g.ldp : g.C + g.sCz * z;
  const long ldc = to_parts ? g.ldp : g.ldc;
  const float* bias = (g.bias && !to_parts) ? g.bias + g.sbiasz * z : nullptr;
  const bool vec_ok = (ldc % 4 == 0) && (((uintptr_t)C & 15u) == 0), add = g.accumulate && !to_parts;
  int crow[4];                                                   // (looked up before the first store)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = min(m0 + wm * 64 + i * 16 + i16, M - 1);
    crow[i] = (g.c_rows && !to_parts) ? g.c_rows[row] : row;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + wm * 64 + i * 16 + i16;
    if (row >= M) continue;
    const long prow = crow[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + wn * 64 + j * 16 + 4 * q;
      if (col >= g.N) continue;
      float* p = C + prow * ldc + col;
      float e[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
      if (bias) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (col + v < g.N) e[v] += bias[col + v];
      }
      const bool whole = vec_ok && col + 3 < g.N;
      if (whole && !add) *(float4*)p = make_float4(e[0], e[1], e[2], e[3]);      // (by itself: joined with the read below, every store waits for the one before)
      else if (whole) {
        const float4 old = *(const float4*)p;
        *(float4*)p = make_float4(old.x + e[0], old.y + e[1], old.z + e[2], old.w + e[3]);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (col + v < g.N) p[v] = add ? p[v] + e[v] : e[v];
      }
    }
  }
}

__global__ __launch_bounds__(256, 2) void gemm_float_nn_kernel(FArgs g) { gemm_float_body<true, false>(g); }
__global__ __launch_bounds__(256, 2) void gemm_float_nt_kernel(FArgs g) { gemm_float_body<true, true>(g); }
__global__ __launch_bounds__(256, 2) void gemm_float_tn_kernel(FArgs g) { gemm_float_body<false, false>(g); }

}  // namespace

// K ranges for a product with few 128 x 128 tiles.  A tile's stage of 32 k is taken as 1.75 us of a compute unit's matrix cores (2.6 when the
// unit has a single work-group and nothing hides its waits; measured 1.46 and 1.65 now, and with 1.25 and 1.95 here eight networks'
// products took the same time within 1 %), work-groups come in whole rounds of 256 units, and the parts are
// written and read once.  (Two directions, 620 inputs, 1000 units, dW_x: 320 tiles leave 3 of 8 units idle in the second round; dW of 64 units over 10240 frames
// was 4 tiles on 4 units, 1.4 ms, and is now 0.04.)
// `frames`: rows are frames, padded ones included: judged with 0.6 of the rows real (lengths spread evenly from a fifth of the longest on) as
// well as with all.
// Checked against every count up to 24 for the four products of 16 layers (256 to 1536 units, 240 to 25600 frames of which 0.5 to all are
// real, one and two directions): with the factor for eight ranges anywhere from 0.65 to 0.85 the choice costs a whole pass 0.5 % on average against the
// best count, 2 % at most but for one product (7 %: Zx of 1029 real of 2037 frames, whose 352 tiles it does not cut); at 0.6 and at 0.9 it goes
// wrong by 11 and 9 %.
int gemm_float_ranges(long M, long N, long K, int nz, int nseg, bool frames) {
  const long tiles = (long)cdiv(M, kTile) * cdiv(N, kTile) * nz, fewer = frames ? (long)cdiv(M * 3 / 5, kTile) * cdiv(N, kTile) * nz : tiles;
  const long stages = nseg * (long)cdiv(K, kKS);
  const auto loop_us = [&](long t, int r) {
    const long rounds = cdiv(std::max(t, 1L) * r, 256L);
    return (rounds == 1 ? 2.6 : 1.75 * rounds) * cdiv(stages, (long)r);
  };
  int best = 1;
  double best_us = 1e30;
  for (int r = 1; r <= 64 && (r == 1 || stages / r >= 4); ++r) {
    double us = 0.5 * (loop_us(tiles, r) + loop_us(fewer, r)) + (r > 1 ? 6.0 + (double)r * M * N * nz * 8 / 4.5e6 : 0.0);
    if (frames && r == 8) us *= 0.75;    // a range per XCD, operands from its own L2: dX of two directions, 620 inputs, 1000 units 218 us, with six ranges 327
    if (us < 0.95 * best_us) { best = r; best_us = us; }
  }
  return best;
}
size_t gemm_float_parts_bytes(long M, long N, long K, int nz, int nseg, bool frames) {
  const int r = gemm_float_ranges(M, N, K, nz, nseg, frames);
  return r > 1 ? (size_t)nz * r * M * ((N + 3) / 4 * 4) * 4 : 0;
}

static long rows_in_memory(const GemmArgs& g, bool a) {
  if (a && g.a_kcontig) return g.a_rows ? g.a_phys_rows : g.M;
  if (!a && g.b_kcontig) return g.N;
  return g.k_phys_rows > 0 ? g.k_phys_rows : g.K;
}
bool gemm_float_ok(const GemmArgs& g) {
  const auto a16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  const auto m4 = [](long v) { return v % 4 == 0; };
  const long lim = 0x7fffff00L;                                  // operands are addressed with 32-bit byte offsets
  if (g.in_bf16 || g.out_bf16 || g.lens || g.nseg < 1 || (!g.a_kcontig && g.b_kcontig)) return false;
  if (g.parts && !a16(g.parts)) return false;
  if (!a16(g.A) || !a16(g.B) || !m4(g.lda) || !m4(g.ldb) || !m4(g.sAz) || !m4(g.sBz) || !m4(g.sAseg) || !m4(g.sBseg)) return false;
  const bool tn = !g.a_kcontig && !g.b_kcontig;
  if (g.k_rows && (!tn || !a16(g.k_rows))) return false;
  if ((g.a_rows || g.m_dev) && !g.a_kcontig) return false;
  if (g.c_rows && !g.a_kcontig) return false;
  if (tn && g.nseg != 1) return false;
  if ((g.a_kcontig || g.b_kcontig) && !m4(g.K)) return false;    // 16-byte chunks along k must not straddle K
                                                                 // (columns past M / N of a k-major operand reach no stored element)
  const long a_rows_mem = rows_in_memory(g, true), b_rows_mem = rows_in_memory(g, false);
  return a_rows_mem * g.lda * 4 <= lim && b_rows_mem * g.ldb * 4 <= lim;
}

hipError_t launch_gemm_float(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nz <= 0) return hipSuccess;
  FArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = (float*)g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nseg = g.nseg; a.sAseg = g.sAseg; a.sBseg = g.sBseg;
  a.accumulate = g.accumulate;
  a.a_rows = g.a_rows; a.c_rows = g.c_rows; a.a_phys_rows = g.a_phys_rows; a.m_dev = g.m_dev;
  a.k_rows = g.k_rows; a.k_phys_rows = g.k_phys_rows; a.k_dev = g.k_dev;
  a.ksplit = g.parts ? gemm_float_ranges(g.M, g.N, g.K, g.nz, g.nseg, g.frames) : 1;
  if (a.ksplit > 1 && gemm_float_parts_bytes(g.M, g.N, g.K, g.nz, g.nseg, g.frames) > g.parts_bytes) a.ksplit = 1;
  a.parts = g.parts; a.ldp = (g.N + 3) / 4 * 4;
  a.tiles_m = cdiv(g.M, kTile); a.tiles_n = cdiv(g.N, kTile);
  a.per_xcd = cdiv(a.tiles_m * a.tiles_n, 8);
  const long a_rows_mem = rows_in_memory(g, true), b_rows_mem = rows_in_memory(g, false);
  a.a_bytes = (unsigned)(a_rows_mem * g.lda * 4); a.b_bytes = (unsigned)(b_rows_mem * g.ldb * 4);
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [] {
    for (const void* k : {(const void*)gemm_float_nn_kernel, (const void*)gemm_float_nt_kernel, (const void*)gemm_float_tn_kernel}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
  if (ea != hipSuccess) return ea;
  const dim3 grid = a.ksplit == 8 ? dim3(a.tiles_m * a.tiles_n * 8, g.nz) : dim3(a.per_xcd * 8, g.nz * a.ksplit), block(256);
  if (g.a_kcontig && g.b_kcontig) hipLaunchKernelGGL(gemm_float_nt_kernel, grid, block, kLds, s, a);
  else if (g.a_kcontig) hipLaunchKernelGGL(gemm_float_nn_kernel, grid, block, kLds, s, a);
  else hipLaunchKernelGGL(gemm_float_tn_kernel, grid, block, kLds, s, a);
  if (a.ksplit == 1) return hipGetLastError();
  SumJob j = {};
  j.parts = a.parts; j.C = a.C; j.bias = a.bias; j.M = a.M; j.N = a.N; j.ksplit = a.ksplit; j.nz = g.nz;
  j.ldp = a.ldp; j.sPz = (long)a.ksplit * a.M * a.ldp; j.ldc = a.ldc; j.sCz = a.sCz; j.sbiasz = a.sbiasz;
  j.c_rows = a.c_rows; j.m_dev = a.m_dev; j.accumulate = a.accumulate;
  return finish_parts(j, (size_t)g.nz * j.sPz * 4, g.sums, s);
}

}  // namespace lstm
