// Fast path of the hoisted matrix products for bfloat16 storage.
//
// gemm_dl8_* (operands loaded straight into LDS, eight wavefronts; described where it is defined):
//     C[M,N] (+)= sum_seg A_seg[M,K] . B_seg[N,K]^T  (+ bias[N]),
// both operands k-contiguous, rows 8-byte aligned, K a multiple of 4: dX = DZ W_x^T of long batches; gemm_nn8: the same with B k-major, Zx = X W_x + b
// with W_x as it lies in memory.
// gemm_tn8_f32: the k-major operand pair of the weight gradients dW_x = X^T DZ, dW_h = Hprev^T DZ.
// Products with fewer 256 x 256 tiles than fill the device are gemm_tile.hip's.
#include "common.h"
#include "recurrent_dev.h"
#include <algorithm>

namespace lstm {
namespace {

constexpr int kT = 256;                   // tile edge (both M and N)
constexpr int kKB = 64;                   // k per stage (bf16 elements)
constexpr int kSupM = 8, kSupN = 4;   // tiles per XCD-resident block (kSupM * kSupN = 32 CUs)

struct NtArgs {
  const char* A; const char* B; void* C; const float* bias;
  int M, N, K;
  int ktail;                              // both operands k-contiguous: four k behind the K (a multiple of 8) that the stages walk
  long lda, ldb, ldc;                     // elements
  long sAz, sBz, sCz, sbiasz; int nz;
  int nseg; long sAseg, sBseg;
  int accumulate;
  const int* a_rows; const int* c_rows;   // logical row -> physical row of A / of C (NULL: identity)
  const int* k_rows; int k_phys_rows;     // k-major kernel: k -> row of A and B in memory (NULL: identity), rows in memory
  const int* m_dev; const int* k_dev;     // device-resident M / K (NULL: use M / K above)
  int a_phys_rows;                        // rows of A in memory when a_rows is given
  int ksplit;                             // k-major kernel: K ranges, each a z of its own (0: one)
  int blocked;                            // tile raster: 1 = blocks of kSupM x kSupN tiles per XCD, 0 = bands of 8 tile columns
};

__device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices

// What every kernel variant needs to know about its tile.
struct TileCoord { int M, K, m0, n0, z, pos; bool live; };
__device__ __forceinline__ TileCoord tile_coord(const NtArgs& g) {
  TileCoord t;
  t.live = false;
  t.pos = 0;                                        // place inside the XCD's block of tiles (blocked raster; else 0)
  t.M = g.m_dev ? min(g.M, *g.m_dev) : g.M;        // the grid is sized for g.M; surplus tiles leave at once
  t.K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  const int tiles_m = (g.M + kT - 1) / kT, tiles_n = (g.N + kT - 1) / kT;
  const int bid = blockIdx.x;
  int tm, tn;
  if (g.blocked) {
    // Work-groups are dealt to the eight XCDs round-robin, so blockIdx & 7 is the XCD and blockIdx >> 3 counts the
    // work-groups of that XCD in launch order.  The 32 work-groups an XCD runs at a time form a block of
    // kSupM x kSupN tiles: kSupM + kSupN operand panels feed kSupM * kSupN tiles out of that XCD's L2.
    const int sup_m = (tiles_m + kSupM - 1) / kSupM, sup_n = (tiles_n + kSupN - 1) / kSupN;
    const int xcd = bid & 7, slot = bid >> 3;
    const int sup = (slot / (kSupM * kSupN)) * 8 + xcd, pos = slot % (kSupM * kSupN);
    if (sup >= sup_m * sup_n) return t;
    const int sn = sup % sup_n, sm = sup / sup_n;
    tm = sm * kSupM + pos / kSupN; tn = sn * kSupN + pos % kSupN;
    t.pos = pos;
    if (tm >= tiles_m || tn >= tiles_n) return t;
  } else {
    // few tiles: bands of 8 tile columns, row-major inside a band; every XCD keeps one B tile column in its L2
    const int band = bid / (8 * tiles_m);
    const int width = min(8, tiles_n - band * 8);
    const int rel = bid - band * 8 * tiles_m;
    tn = band * 8 + rel % width; tm = rel / width;
  }
  t.m0 = tm * kT; t.n0 = tn * kT;
  if (t.m0 >= t.M) return t;
  t.z = blockIdx.y;
  t.live = true;
  return t;
}

// Writes a work-group's 256x256 accumulator tile to C.  The tile is held by 2 x (8 / TN) wavefronts, each
// 4 x TN MFMA blocks of 32x32 (TN = 4: 2x2 wavefronts of 128x128; TN = 2: 2x4 wavefronts of 128x64).
template <typename TC, int TN, bool SPREAD = false>           // SPREAD: the wavefronts' 32-column blocks alternate (block j of all of them, then j + 1)
__device__ __forceinline__ void store_tile(f32x16 (&acc)[4][TN], char* lds, const NtArgs& g, int M, int m0, int n0, int z) {
  constexpr int WN = 8 / TN, NW = 2 * WN;            // wavefronts along N, wavefronts in all
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;     // (uniform: rows of C are looked up by scalar loads)
  const int wm = wave / WN, wn = wave % WN;
  const int r = lane & 31, gq = lane >> 5;
  const auto col_of = [&](int j) { return SPREAD ? j * (WN * 32) + wn * 32 + r : wn * (TN * 32) + j * 32 + r; };
  // Epilogue.  A lane holds column (lane % 32), rows 8*(v/4) + 4*(lane/32) + v%4 of each 32x32 block: stored as
  // it is that would be 128-byte pieces, eight of them per row at different times.  The tile goes through LDS
  // instead (two halves of 128 rows, the main loop's buffers are free by now) and leaves as whole rows: one
  // wavefront store = 256 consecutive columns of one row.
  TC* C = (TC*)g.C + g.sCz * z;
  const float* bias = g.bias ? g.bias + g.sbiasz * z : nullptr;
  constexpr int kEpStride = 260;                      // floats per staged row (16-byte aligned, off the bank period)
  float* ep = (float*)lds;
  const bool vec_ok = (g.ldc % 4 == 0) && (((uintptr_t)C & 15u) == 0);
  float bv[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + col_of(j);
    bv[j] = (bias && col < g.N) ? bias[col] : 0.f;
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();                                   // LDS free: main loop done / previous half stored
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rowl = wm * 64 + ii * 32 + 8 * (v >> 2) + 4 * gq + (v & 3);
          ep[rowl * kEpStride + col_of(j)] = acc[2 * half + ii][j][v] + bv[j];
        }
    __syncthreads();
    const int col = n0 + lane * 4;
    for (int rr = 0; rr < 128 / NW; ++rr) {
      const int rowl = wave * (128 / NW) + rr;
      const int row = m0 + (rowl >> 6) * 128 + half * 64 + (rowl & 63);
      if (row >= M) break;                             // rows ascend with rr inside a wave's share
      if (col >= g.N) continue;
      const float4 val = *(const float4*)&ep[rowl * kEpStride + lane * 4];
      const float e[4] = {val.x, val.y, val.z, val.w};
      const long off = (long)(g.c_rows ? g.c_rows[row] : row) * g.ldc + col;
      const bool whole = vec_ok && col + 3 < g.N;
      if constexpr (sizeof(TC) == 4) {
        float* Cf = (float*)C + off;
        const bool add = g.accumulate;
        // (by itself: joined with the read below, every row waits for the one before; non-temporal: the operand panels stay in L2)
        if (whole && !add) __builtin_nontemporal_store((f32x4){val.x, val.y, val.z, val.w}, (f32x4*)Cf);
        else if (whole) {
          const float4 old = *(const float4*)Cf;
          *(float4*)Cf = make_float4(val.x + old.x, val.y + old.y, val.z + old.z, val.w + old.w);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (col + k < g.N) Cf[k] = add ? Cf[k] + e[k] : e[k];
        }
      } else {
        uint16_t* Cb = (uint16_t*)C + off;
        if (whole) {
          uint2 o;
          o.x = f2bf_bits(e[0]) | ((unsigned)f2bf_bits(e[1]) << 16);
          o.y = f2bf_bits(e[2]) | ((unsigned)f2bf_bits(e[3]) << 16);
          *(uint2*)Cb = o;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (col + k < g.N) Cb[k] = f2bf_bits(e[k]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// Same product with the operands brought from global memory straight into LDS (16-byte-per-lane buffer loads
// with the LDS destination: no staging registers, no LDS store instructions), for K a multiple of 64.
//
// LDS holds two stages of [A | B], each operand 256 rows of 128 bytes (64 bf16), unpadded: a wavefront-wide
// load fills 1 KiB = 8 consecutive rows, lane l writing bytes 16*l of it.  Bank conflicts of the fragment reads
// are avoided by the placement instead of padding: the 16-byte slot p of row r holds k-chunk p ^ ((r >> 1) & 7),
// which the loading lane arranges by choosing WHICH global chunk it fetches.
//
// Eight wavefronts (2 x 4) of 128x64 = 4 x 2 MFMA blocks, two per SIMD, so one wavefront's LDS reads and waits hide behind the
// other's MFMAs (four wavefronts of 128x128 measured 15-20 % slower).  A stage (k advances 64) is four phases, a quarter of the
// wavefront's blocks each over all 64 k: blocks (rows 0-1, column 0), (0-1, 1), (2-3, 1), (2-3, 0).  A phase reads the fragments it lacks
// - A's first half and B's first, B's second, A's second, none -, meets the others, multiplies, meets them again; wavefronts 4-7 are
// half a phase behind, so that on every SIMD one wavefront multiplies while the other reads.  A half of an operand is free for the stage
// after next as soon as all have read it, and its two wavefront-loads go out in the next phase: every load has six or seven phases
// to arrive, 80 to 96 KiB are always on their way, and no wait ever drains them (vmcnt(10)).
// Before, a stage's loads went out together and were waited for together, a stage later, at a barrier all wavefronts met at once: 8192^3
// 1137 TFLOP/s, 24576 x 2048 x 8192 1121, 27136 x 8192 x 2048 (float C) 1074, 3200 x 8000 x 2000 771; now 1208, 1252, 1136, 857 (without
// the half phase between the wavefronts 1083, 1082, 1021, 740).  On zeros 8192^3 runs at 1680: what is left is the clock, which the
// data's switching brings down to about 1.7 GHz, and where N is small the loads (without MFMAs 24576 x 2048 x 8192 takes the same time).
constexpr int kDlRow = 128;                  // bytes per LDS row
constexpr int kDlOp = kT * kDlRow;           // one operand, one stage (32 KiB)
constexpr int kDlStage = 2 * kDlOp;
constexpr int kDlLds = 133120;               // max(two stages, the epilogue's staging of 128 rows x 260 floats)
// A buffer load whose data goes to LDS (M0 = wavefront-uniform LDS byte address; lane l writes M0 + size * l) instead of
// registers.  Written as assembly on purpose: the compiler makes every later LDS read wait for ALL such loads
// it knows to be in flight (it cannot tell that they fill the other stage), which would serialise loads and MFMAs.
// The kernel orders them itself with explicit vmcnt waits and barriers.  Nothing else in these kernels uses M0.
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

//
// BROWS: B lies k-major (W_x as the caller holds it: transposing it first took 17 us of 32 MB, a sixth of the product with 3200 rows).  Half h of a stage of B
// is then 64 k-rows of columns 128 h .. + 127 (256 bytes in a row, four rows a wavefront-load), the wavefronts' blocks lie accordingly (store_tile: SPREAD),
// and fragments leave LDS through the transpose read, its 64-byte blocks of row k XORed with k % 4 (see gemm_tn_body).
template <typename TC, bool RAGGED, bool BROWS = false>
__device__ __forceinline__ void gemm_dl_body(const NtArgs& g) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int TN = 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int r = lane & 31, gq = lane >> 5;

  const TileCoord tc = tile_coord(g);
  if (!tc.live) return;
  const int M = tc.M, K = tc.K, m0 = tc.m0, n0 = tc.n0, z = tc.z;

  f32x16 acc[4][TN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  if (!BROWS && g.ktail) {
    for (int seg = 0; seg < g.nseg; ++seg) {
      uint2 ta[4], tb[TN];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = m0 + wm * 128 + i * 32 + r;
        ta[i] = make_uint2(0u, 0u);
        if (gq == 0 && row < M) ta[i] = *(const uint2*)(g.A + (g.sAz * z + g.sAseg * seg + (long)(g.a_rows ? g.a_rows[row] : row) * g.lda + K) * 2);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = n0 + wn * 64 + j * 32 + r;
        tb[j] = make_uint2(0u, 0u);
        if (gq == 0 && row < g.N) tb[j] = *(const uint2*)(g.B + (g.sBz * z + g.sBseg * seg + (long)row * g.ldb + K) * 2);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mma_last4(ta[i], tb[j], acc[i][j]);
    }
  }

  // K is a multiple of 8 (whole 16-byte chunks).  The last k-tile of a segment may hold fewer than 8 chunks: the lanes
  // that would fetch a chunk past K point outside the buffer descriptor for that tile and their slots arrive as zeros.
  const int ktiles = (K + kKB - 1) / kKB;
  const int tail_chunks = (K - (ktiles - 1) * kKB) >> 3;       // 1 .. 8 chunks in the last k-tile
  const bool ragged = RAGGED && tail_chunks < 8;              // RAGGED = false: the launcher saw K % 64 == 0
  const int total = ktiles * g.nseg;                           // stages

  // Loads.  A quarter of a stage (two wavefront-loads of every wavefront) is half an operand: rows of every wavefront's first or second
  // two (A) or one (B) MFMA blocks.  Wavefront-load j of it fills 8 rows; lane l fills slot l & 7 of row l >> 3 of those, i.e. fetches
  // k-chunk (l & 7) ^ swizzle(row).  Rows past the operand's end point outside the buffer descriptor and arrive as zeros.
  const int chunk = (lane & 7) ^ ((((wave & 1) * 8 + (lane >> 3)) >> 1) & 7);
  const bool past = chunk >= tail_chunks;                      // this lane's chunk lies past K in a ragged last k-tile
  const int b_row = wave * 4 + (lane >> 4), b_col = ((((lane >> 2) & 3) ^ (lane >> 4)) * 32) + (lane & 3) * 8;      // BROWS: of load 0 of a half (load 1: 32 rows on)
  const int b_tail = (g.k_phys_rows ? g.k_phys_rows : K) - (ktiles - 1) * kKB;      // BROWS: rows of B in the last k-tile
  unsigned vo[2][2][2], lrow[2][2][2];                         // [operand][half][load]
  const long a_rows_mem = g.a_rows ? g.a_phys_rows : M;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int ta = j * 128 + h * 64 + wave * 8, tb = (j * 2 + (wave >> 2)) * 64 + h * 32 + (wave & 3) * 8;
      lrow[0][h][j] = ta * kDlRow; lrow[1][h][j] = kDlOp + tb * kDlRow;
      long ra = m0 + ta + (lane >> 3), rb = n0 + tb + (lane >> 3);
      if (g.a_rows) ra = ra < M ? (long)g.a_rows[ra] : 0x7fffffffL; else if (ra >= M) ra = 0x7fffffffL;
      if (rb >= g.N) rb = 0x7fffffffL;
      const long oa = (ra * g.lda) * 2 + chunk * 16, ob = (rb * g.ldb) * 2 + chunk * 16;
      vo[0][h][j] = (ra >= a_rows_mem || oa > 0x7ffffff0L) ? 0x7ffffff0u : (unsigned)oa;
      vo[1][h][j] = (rb >= g.N || ob > 0x7ffffff0L) ? 0x7ffffff0u : (unsigned)ob;
      if constexpr (BROWS) {
        lrow[1][h][j] = kDlOp + h * (kDlOp / 2) + (j * 8 + wave) * 1024;
        const int col = n0 + h * 128 + b_col;
        vo[1][h][j] = col < g.N ? (unsigned)(((long)(b_row + j * 32) * g.ldb + col) * 2) : 0x7ffffff0u;
      }
    }
  const long a_bytes = a_rows_mem * g.lda * 2, b_bytes = (long)(BROWS ? (g.k_phys_rows ? g.k_phys_rows : K) : g.N) * g.ldb * 2;
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;
  const unsigned rec[2] = {a_bytes > 0x7fffffffL ? 0x7fffffffu : (unsigned)a_bytes, b_bytes > 0x7fffffffL ? 0x7fffffffu : (unsigned)b_bytes};
  const char* const base[2] = {g.A + g.sAz * z * 2, g.B + g.sBz * z * 2};
  const long seg_bytes[2] = {g.sAseg * 2, g.sBseg * 2};
  struct Stage { int it, seg, kt; };                           // a stage whose loads go out
  auto advance = [&](Stage& t) __attribute__((always_inline)) {
    ++t.it;
    if (++t.kt == ktiles) { t.kt = 0; ++t.seg; }
  };
  // (past the last stage the same loads are issued with every lane outside the descriptor: the counted waits below count them)
  auto issue = [&](const Stage& t, int op, int h) __attribute__((always_inline)) {
    const u32x4 rs = make_rsrc(base[op] + seg_bytes[op] * t.seg, t.it < total ? rec[op] : 0u);
    const unsigned dst = lds_base + (t.it & 1) * kDlStage, koff = t.kt * (kKB * 2);
    const bool cut = ragged && t.kt == ktiles - 1;
    if (BROWS && op == 1) {
      const unsigned boff = (unsigned)t.kt * (unsigned)g.ldb * (kKB * 2u);
      const int rows = RAGGED && t.kt == ktiles - 1 ? b_tail : kKB;
#pragma unroll
      for (int j = 0; j < 2; ++j) load_to_lds_b128(rs, dst + lrow[op][h][j], RAGGED && b_row + j * 32 >= rows ? 0x7ffffff0u : vo[op][h][j], boff);
      return;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) load_to_lds_b128(rs, dst + lrow[op][h][j], (cut && past) ? 0x7ffffff0u : vo[op][h][j], koff);
  };

  // Fragment reads: row (wm*128 + i*32 + r) of A / (wn*64 + j*32 + r) of B, k-chunk 2*s + gq, which sits in
  // slot (2*s + gq) ^ ((r >> 1) & 7): one XOR with s * 32 per k-step on a per-lane base offset.
  const int fa_off = (wm * 128 + r) * kDlRow + ((gq ^ ((r >> 1) & 7)) * 16);
  const int fb_off = kDlOp + (wn * 64 + r) * kDlRow + ((gq ^ ((r >> 1) & 7)) * 16);
  const int ft_off = kDlOp + (gq * 8 + ((lane & 15) >> 2)) * 256 + ((wn ^ ((lane & 15) >> 2)) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;     // BROWS
  uint4 fa[2][4], fb[TN][4];                                   // [block][k-step]
  auto read_a = [&](int it, int h) __attribute__((always_inline)) {
    const char* p = lds + (it & 1) * kDlStage;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s = 0; s < 4; ++s) fa[i][s] = *(const uint4*)(p + (fa_off ^ (s * 32)) + (2 * h + i) * 32 * kDlRow);
  };
  auto read_b = [&](int it, int j) __attribute__((always_inline)) {
    const char* p = lds + (it & 1) * kDlStage;
    if constexpr (BROWS) {
      typedef __attribute__((ext_vector_type(4))) short s16x4;
      const auto turned = [](const char* q) { return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)q)); };
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint2 lo = turned(p + ft_off + j * (kDlOp / 2) + s * 4096), hi = turned(p + ft_off + j * (kDlOp / 2) + s * 4096 + 1024);
        fb[j][s] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
      return;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) fb[j][s] = *(const uint4*)(p + (fb_off ^ (s * 32)) + j * 32 * kDlRow);
  };
  // The end of a phase's reading half: this wavefront's reads have returned (what they read may be overwritten once all have met), and
  // the quarter that the next phase reads has landed (ten younger loads).
  auto meet = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  auto multiply = [&](int h, int j) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x007a);                        // vmcnt(10) lgkmcnt(0)
    meet();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[2 * h + i][j] = mma(fa[i][s], fb[j][s], acc[2 * h + i][j]);
    __builtin_amdgcn_s_setprio(0);
    meet();
  };

  if (total > 0) {
    Stage nx = {0, 0, 0};
    issue(nx, 0, 0); issue(nx, 1, 0); issue(nx, 1, 1); issue(nx, 0, 1);
    advance(nx);
    issue(nx, 0, 0); issue(nx, 1, 0); issue(nx, 1, 1);
    __builtin_amdgcn_s_waitcnt(0x0f7a);                        // vmcnt(10): the first stage's first halves
    meet();
    if (wm == 1) meet();                                       // the second four wavefronts stay half a phase behind
    for (int it = 0; it < total; ++it) {
      read_a(it, 0); read_b(it, 0);
      issue(nx, 0, 1);                                         // stage it + 1
      advance(nx);                                             // stage it + 2, into this stage's buffer
      multiply(0, 0);
      read_b(it, 1);
      issue(nx, 0, 0);
      multiply(0, 1);
      read_a(it, 1);
      issue(nx, 1, 0);
      multiply(1, 1);
      issue(nx, 1, 1);
      multiply(1, 0);
    }
    if (wm == 0) meet();
    __builtin_amdgcn_s_waitcnt(0x0f70);                        // vmcnt(0): the epilogue uses LDS
  }
  store_tile<TC, TN, BROWS>(acc, lds, g, M, m0, n0, z);
}

// ---------------------------------------------------------------------------------------------------------
// The weight-gradient shape, C[M,N] = sum_k A[k][m] B[k][n] with BOTH operands stored k-major (a row per frame:
// dW_x = X^T DZ, dW_h = Hprev^T DZ; float C), without transposing anything in memory.  Same tile, wavefront
// layout and epilogue as gemm_dl_body; what differs is how a stage sits in LDS and how MFMA
// fragments leave it:
//   * a stage is 64 k-rows of 256 columns (512 bytes) per operand; a wavefront-load brings two whole rows (full
//     lines).  Row k may be any row of the operand in memory (`k_rows`: the packed list of real frames), looked up
//     one stage ahead of the load that needs it;
//   * MFMA wants, per lane, 8 consecutive k of ONE column, which in a k-major tile are 512 bytes apart.  The LDS
//     transpose read (8 bytes per lane, 16-bit elements) does that turn inside each group of 16 lanes: lane s
//     supplies the address of row kbase + s/4, columns cbase + 4*(s%4) .. +3, and lane l receives column cbase + l
//     of rows kbase .. kbase+3 (layout measured on the device).  Two such reads make one MFMA operand;
//   * the four rows a 16-lane group reads together lie 512 bytes apart, i.e. in the same banks; so the 64-byte
//     blocks of row k are stored XORed with k % 4 (again by choosing which global chunk a loading lane fetches).
// A stage is four phases, one k-step of all eight blocks each, run as in gemm_dl_body: reads, meeting, products, meeting, with four of the
// wavefronts half a phase behind.  Sixteen k-rows of both operands are one wavefront-load per operand and wavefront; their place is free for the
// stage after next once all have read them, so they go out in the next phase and have seven phases to arrive, 112 KiB on their way.
// Before, a stage's loads went out between the products of one k-step and were waited for a stage later, at a barrier all wavefronts met at once: dW_x of 31597
// frames (2048 x 4096, two directions) 987 TFLOP/s, of 3054 (2000 x 4000) 801; now 1226 and 953.
template <typename TC, bool ROWS, bool RANGES>                 // ROWS: the k-rows are those of a list (k_rows); RANGES: K in ksplit ranges
__device__ __forceinline__ void gemm_tn_body(const NtArgs& g) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int TN = 2, WN = 4, NW = 8, NS = 4;                // 8 wavefronts of 128x64; k-steps of a stage = wavefront-loads per operand
  constexpr int kRow = 512;                                    // bytes per k-row of a stage (256 columns)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  const TileCoord tc = tile_coord(g);
  if (!tc.live) return;
  const int M = tc.M, K = tc.K, m0 = tc.m0, n0 = tc.n0, ks = RANGES ? g.ksplit : 1, z = RANGES ? tc.z / ks : tc.z;

  f32x16 acc[4][TN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int stages = (K + kKB - 1) / kKB, each = (stages + ks - 1) / ks, first = RANGES ? (tc.z - z * ks) * each : 0;       // rows past K arrive as zeros
  const int total = RANGES ? min(each, stages - first) : stages;         // this range's (0 or less: its part is zeros)

  // Loads.  The wavefront-load of k-step q fills k-rows 2*(q*NW + wave) and +1 of the stage; lane l fills
  // 16-byte slot l % 32 of row l / 32, i.e. fetches column chunk (l % 32) ^ 4*(k % 4).
  const int krow_in_stage = 2 * wave + (lane >> 5);            // + 2*NW*q
  const int chunk = (lane & 31) ^ (4 * (krow_in_stage & 3));   // 2*NW*q is a multiple of 4
  const bool a_col_ok = m0 + chunk * 8 < M, b_col_ok = n0 + chunk * 8 < g.N;
  const unsigned a_col = (m0 + chunk * 8) * 2, b_col = (n0 + chunk * 8) * 2, lda2 = (unsigned)g.lda * 2, ldb2 = (unsigned)g.ldb * 2;
  const unsigned rows_mem = ROWS ? (unsigned)g.k_phys_rows : (unsigned)K;
  const long a_bytes = (long)rows_mem * g.lda * 2, b_bytes = (long)rows_mem * g.ldb * 2;
  const unsigned a_rec = a_bytes > 0x7fffffffL ? 0x7fffffffu : (unsigned)a_bytes, b_rec = b_bytes > 0x7fffffffL ? 0x7fffffffu : (unsigned)b_bytes;
  const u32x4 ra = make_rsrc(g.A + g.sAz * z * 2, a_rec), rb = make_rsrc(g.B + g.sBz * z * 2, b_rec);
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;
  // Memory rows of the stage whose loads go out next.  A wavefront-load covers rows k and k+1 of the list, the same
  // for all lanes of a half, so the look-up is a scalar load of two consecutive entries - written as assembly and
  // waited for by hand, a phase later: the compiler would wait for a look-up it knows about right where it is issued, and with vector loads
  // that wait would also cover every operand load in flight.  The list must be readable up to the next multiple of 64 entries.
  typedef __attribute__((ext_vector_type(2))) int i32x2;
  i32x2 prow[NS];
  auto lookup = [&](int it) __attribute__((always_inline)) {
    if constexpr (ROWS) {
      const int* p = g.k_rows + (long)(first + min(it, total - 1)) * kKB + 2 * wave;        // (past the last stage `issue` looks at no row)
#pragma unroll
      for (int q = 0; q < NS; ++q) asm volatile("s_load_dwordx2 %0, %1, %2" : "=s"(prow[q]) : "s"(p), "n"(q * 2 * NW * 4) : "memory");
    }
  };
  auto looked_up = [&]() __attribute__((always_inline)) {
    if constexpr (ROWS) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(prow[0]), "+s"(prow[1]), "+s"(prow[2]), "+s"(prow[3])::"memory");
  };
  // (past K, also past the last stage, with every lane outside the descriptor: the counted waits below count these loads)
  auto issue = [&](int it, int q) __attribute__((always_inline)) {
    const unsigned dst = lds_base + (it & 1) * kDlStage + (q * NW + wave) * 1024;
    const int k = RANGES && it >= total ? K : (first + it) * kKB + 2 * NW * q + krow_in_stage;
    const int row = ROWS ? ((lane >> 5) ? prow[q][1] : prow[q][0]) : k;
    const bool row_ok = (k < K) & ((unsigned)row < rows_mem);
    const unsigned oa = (unsigned)row * lda2 + a_col, ob = (unsigned)row * ldb2 + b_col;           // (below 2^31: gemm_tn_ok)
    load_to_lds_b128(ra, dst, (row_ok & a_col_ok) ? oa : 0x7ffffff0u, 0);
    load_to_lds_b128(rb, dst + kDlOp, (row_ok & b_col_ok) ? ob : 0x7ffffff0u, 0);
  };

  // Fragment reads (see the head of this function).  Lane L = 32*kg + 16*grp + l: source row kg*8 + l/4 (+4 for the
  // second read) of the 16-row k-step, columns block*32 + grp*16 + 4*(l%4) .. +3, 64-byte blocks XORed with row % 4.
  const int l16 = lane & 15, grp = (lane >> 4) & 1, kg = lane >> 5;
  const int fr_row = (kg * 8 + (l16 >> 2)) * kRow, fr_sw = (l16 >> 2) & 3, fr_low = grp * 32 + (l16 & 3) * 8;
  int fa_off[4], fb_off[TN];
#pragma unroll
  for (int i = 0; i < 4; ++i) fa_off[i] = fr_row + ((((wm * 4 + i) ^ fr_sw) & 7) << 6) + fr_low;          // column block wm*4 + i of 8
#pragma unroll
  for (int j = 0; j < TN; ++j) fb_off[j] = kDlOp + fr_row + ((((wn * TN + j) ^ fr_sw) & 7) << 6) + fr_low;
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  uint4 fa[4], fb[TN];
  auto tr_read = [&](const char* p) __attribute__((always_inline)) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * kRow));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    return make_uint4(l2.x, l2.y, h2.x, h2.y);
  };
  auto read_frags = [&](int it, int s) __attribute__((always_inline)) {
    const char* base = lds + (it & 1) * kDlStage + s * 16 * kRow;
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = tr_read(base + fa_off[i]);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = tr_read(base + fb_off[j]);
  };
  auto meet = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  // The end of a phase's reading half: its reads have returned, and the loads of the next phase's k-step have landed (twelve younger ones).
  auto end_of_reads = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x007c);                        // vmcnt(12) lgkmcnt(0)
    meet();
  };
  auto multiply = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = mma(fa[i], fb[j], acc[i][j]);
    __builtin_amdgcn_s_setprio(0);
    meet();
  };

  if (total > 0) {
    lookup(0);
    looked_up();
#pragma unroll
    for (int q = 0; q < NS; ++q) issue(0, q);
    lookup(1);
    looked_up();
#pragma unroll
    for (int q = 0; q < 3; ++q) issue(1, q);
    __builtin_amdgcn_s_waitcnt(0x0f7c);                        // vmcnt(12): the first k-step's
    meet();
    if (wm == 1) meet();                                       // the second four wavefronts stay half a phase behind
    for (int it = 0; it < total; ++it) {
      read_frags(it, 0);
      issue(it + 1, 3);
      end_of_reads();
      lookup(it + 2);
      multiply();
      read_frags(it, 1);
      looked_up();
      issue(it + 2, 0);
      end_of_reads();
      multiply();
      read_frags(it, 2);
      issue(it + 2, 1);
      end_of_reads();
      multiply();
      read_frags(it, 3);
      issue(it + 2, 2);
      end_of_reads();
      multiply();
    }
    if (wm == 0) meet();
    __builtin_amdgcn_s_waitcnt(0x0f70);                        // vmcnt(0): the epilogue uses LDS
  }
  store_tile<TC, TN>(acc, lds, g, M, m0, n0, tc.z);
}
template <bool ROWS, bool RANGES> __global__ __launch_bounds__(512, 1) void gemm_tn8_f32_kernel(NtArgs g) { gemm_tn_body<float, ROWS, RANGES>(g); }

// (kernels with literal launch bounds: a bound that depends on a template parameter loses the host-side stub)
template <bool RAGGED> __global__ __launch_bounds__(512, 1) void gemm_dl8_f32_kernel(NtArgs g) { gemm_dl_body<float, RAGGED>(g); }
template <bool RAGGED> __global__ __launch_bounds__(512, 1) void gemm_nn8_f32_kernel(NtArgs g) { gemm_dl_body<float, RAGGED, true>(g); }
template <bool RAGGED> __global__ __launch_bounds__(512, 1) void gemm_dl8_bf16_kernel(NtArgs g) { gemm_dl_body<uint16_t, RAGGED>(g); }

// Frame map of a batch of end-padded sequences: frame (t, b) is kept iff t < lens[b].  Kept frames are numbered
// in (t, b) order: fidx[number] = t*B + b, count[0] = how many are kept,
// count[1] = count[0] rounded up to a multiple of 64.  One wavefront per time step.
__global__ __launch_bounds__(256) void frame_map_kernel(const int* lens, int T, int B, int* fidx, int* count) {
  frame_map_body(blockIdx.x, lens, T, B, fidx, count);
}

__global__ void pad_rows_kernel(const uint16_t* src, uint4* dst, long R, int C, int ldd8) {
  pad_rows_body((long)blockIdx.x * blockDim.x + threadIdx.x, src, dst, R, C, ldd8);
}

}  // namespace

// Rows need not be whole 16 bytes: a load of 16 bytes into LDS wants an address that is a multiple of 4, and where a row of a k-major operand ends inside
// one, what it brings of the next row ends in columns that are not stored.  Rows of 8 n bytes (W_x, DZ) are multiples of 8 whatever n is.
bool gemm_nt_ok(const GemmArgs& g) {
  const auto a8 = [](const void* p) { return ((uintptr_t)p & 7u) == 0; };
  const long lim = 0x7fffff00L;     // operands are addressed with 32-bit byte offsets
  if ((long)g.M * g.lda * 2 > lim || (long)g.N * g.ldb * 2 > lim) return false;
  if (g.k_dev && g.K % 64 != 0) return false;     // a device-resident K counts whole 64-wide stages
  return g.in_bf16 && g.a_kcontig && g.b_kcontig && !g.lens && g.K >= 8 && g.K % 4 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 &&
         g.sAz % 4 == 0 && g.sBz % 4 == 0 && g.sAseg % 4 == 0 && g.sBseg % 4 == 0 && a8(g.A) && a8(g.B);
}

// B k-major, as gemm_nt_ok otherwise (one segment, float C)
bool gemm_nn_ok(const GemmArgs& g) {
  const auto a8 = [](const void* p) { return ((uintptr_t)p & 7u) == 0; };
  const long lim = 0x7fffff00L;     // operands are addressed with 32-bit byte offsets
  if ((long)g.M * g.lda * 2 > lim || ((long)g.K + kKB) * g.ldb * 2 > lim) return false;
  return g.in_bf16 && !g.out_bf16 && g.a_kcontig && !g.b_kcontig && !g.lens && !g.k_dev && !g.k_rows && g.nseg == 1 && g.K % 8 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 &&
         g.N % 4 == 0 && g.sAz % 4 == 0 && g.sBz % 4 == 0 && a8(g.A) && a8(g.B) && (!g.k_phys_rows || (g.k_phys_rows <= g.K && g.K - g.k_phys_rows < kKB));
}

// B k-major: on tiles of 256 x 256 (256 of them at a time) rather than 128 x 128?  us there / here, operands from memory.  Few tiles, gemm_tile_small: there.
// One row of tiles of 128, or one column: there, where no tile is half empty: 64 x 60000 x 256 16 / 25, x 2048 55 / 64, 128 x 200000 x 768 94 / 110, 60000 x 128 x 256 17 / 21.
// A second round at most half full: there while K is short, how short hangs on what neighbours share.  About as many rows as columns, or more: 3300 x 5600 x 1024 64 / 69,
// 9000 x 2048 x 1024 62 / 72, x 2048 101 / 113, but 6000 x 4000 x 2048 125 / 121.  Wider, or fewer than 16 tiles of 128 one way: 1772 x 11120 x 640 49 / 55, 1300 x 13000 x 640 46 / 54,
// 18000 x 1000 x 640 53 / 58, but 2000 x 10000 x 1024 73 / 69, 20000 x 1024 x 1024 73 / 71.  Fewer than 8: 700 x 25000 x 256 37 / 40, x 640 57.4 / 56.9, 640 x 30000 x 256 (354 tiles, 83 % full)
// 32 / 34, x 320 40 / 38, 500 x 45000 x 256 (352, full) 49 / 43; but with a quarter of the larger tiles empty at any K: 300 x 40000 x 640 44 / 51, x 2048 90 / 104.
// A third at most half full: 4100 x 8000 x 256 (544 tiles) 47 / 49, 10000 x 4000 x 256 (640) 53 / 57, but x 1024 106 / 101, and 2000 x 19000 x 128 60 / 58.
// One or two stages of K are little more than storing C: a third or fourth round, and a second that is full, there only where rows of C are whole runs of 64 bytes (more tiles cut more of
// them): 8192 x 4096 x 128 (512 tiles) 38 / 43, 380 x 60000 x 128 (470, a quarter empty) 29 / 32, 6400 x 7680 x 128 (750) 52 / 60, 5683 x 9152 x 128 (828) 58 / 63, 14055 x 4176 x 128 (935)
// 69 / 75; but 5120 x 5632 x 128 (440) 35 / 34, 4000 x 16384 x 128 (1024) 74 / 63, and with rows that are not 6280 x 7560 x 128 (750) 75 / 65, 4097 x 7112 x 40 (476) 47 / 42.
// With the number of rows on the device the host cannot count rounds: here (a forward pass of 60 x 50 frames, half of them real, n_in = 620, n = 1000, both directions, 184 / 176).
bool gemm_nn_pays(const GemmArgs& g) {
  const long tiles = (long)cdiv(g.M, kT) * cdiv(g.N, kT) * g.nz;
  if (gemm_tile_small(g.M, g.N, g.nz) || g.M <= kT / 2 || g.N <= kT / 2) return false;
  if (g.m_dev || tiles <= 256) return true;
  const long m = cdiv(g.M, kT / 2), n = cdiv(g.N, kT / 2), few = std::min(m, n), filled = 25 * m * n * g.nz / tiles;      // percent of the larger tiles that is not padding
  if (tiles <= 384) {
    if (filled <= 75) return false;
    return g.K > (few < 8 ? (tiles <= 320 || filled <= 85 ? 256 : 0) : few >= 16 && n < 2 * m ? 1024 : 640);
  }
  if (tiles > 512 && tiles <= 640 && n < 8 * m) return g.K > 320;
  const bool whole = (long)g.ldc * (g.out_bf16 ? 2 : 4) % 64 == 0 && g.K <= 128;
  if (tiles <= 512) return !(whole && (filled <= 75 || (tiles >= 490 && m >= n)));
  return !(whole && tiles >= 736 && tiles <= 940 && n < 8 * m);
}

bool gemm_tn_ok(const GemmArgs& g) {
  const auto a8 = [](const void* p) { return ((uintptr_t)p & 7u) == 0; };
  const long lim = 0x7fffff00L;     // operands are addressed with 32-bit byte offsets
  const long rows = g.k_rows ? g.k_phys_rows : g.K;
  if (rows * g.lda * 2 > lim || rows * g.ldb * 2 > lim) return false;
  return g.in_bf16 && !g.out_bf16 && !g.a_kcontig && !g.b_kcontig && !g.lens && g.nseg == 1 && !g.a_rows && !g.c_rows && !g.m_dev &&
         g.lda % 4 == 0 && g.ldb % 4 == 0 && g.sAz % 4 == 0 && g.sBz % 4 == 0 && a8(g.A) && a8(g.B);
}

namespace {
hipError_t launch_tn(const GemmArgs& g, int ks, hipStream_t s) {
  NtArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz; a.nseg = 1;
  a.accumulate = g.accumulate; a.k_dev = g.k_dev; a.k_rows = g.k_rows; a.k_phys_rows = g.k_phys_rows;
  if (ks > 1) {
    a.ksplit = ks; a.nz = g.nz * ks; a.accumulate = false; a.bias = nullptr;
    a.C = g.parts; a.ldc = (g.N + 3) / 4 * 4; a.sCz = (long)g.M * a.ldc;
  }
  const int sups = cdiv(cdiv(g.M, kT), kSupM) * cdiv(cdiv(g.N, kT), kSupN);
  a.blocked = sups >= 32 ? 1 : 0;
  const int tiles = a.blocked ? cdiv(sups, 8) * 8 * kSupM * kSupN : cdiv(g.M, kT) * cdiv(g.N, kT);
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [] {
    for (const void* k : {(const void*)gemm_tn8_f32_kernel<false, false>, (const void*)gemm_tn8_f32_kernel<true, false>,
                          (const void*)gemm_tn8_f32_kernel<false, true>, (const void*)gemm_tn8_f32_kernel<true, true>}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kDlLds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
  if (ea != hipSuccess) return ea;
  const auto whole = g.k_rows ? gemm_tn8_f32_kernel<true, false> : gemm_tn8_f32_kernel<false, false>;
  const auto ranged = g.k_rows ? gemm_tn8_f32_kernel<true, true> : gemm_tn8_f32_kernel<false, true>;
  hipLaunchKernelGGL(ks > 1 ? ranged : whole, dim3(tiles, a.nz), dim3(512), kDlLds, s, a);
  return hipGetLastError();
}
// Products of few tiles whose K is long (dW_h of a long batch): as many K ranges as fill the device, at least seven eighths of it, with tiles of which no more than
// a tenth lies outside C; the others stay with the 128 x 128 tiles of gemm_tile.hip.  Parts of the whole device are 64 MiB, written and read, 30 us, so K has to be long.  Both
// sides, dW_x (of 2 n inputs) and dW_h of two directions together, sums included, us: 5744 real of 9600 frames 273 there and 288 here for n = 1024; 12800 of 12800 586
// and 579 (n = 1000 595 and 582, 960 552 and 546); 15344 of 25600 701 and 682; 28784 of 48000 1288 and 1230 (1332 and 1230, 1219 and 1171).  K counts padded frames
// too: with 6144 of them a range n = 1024 begins at 12288.  Widths it leaves out, 28784 frames: 768 (three ranges of 72 tiles) 909 and 1136, 896 1350 and 1279,
// 832 1313 and 1298; 640 and 704, whose tiles lie a sixth outside C, would gain from 12800 frames on (344 and 302, 374 and 340; 28784: 871 and 682, 885 and 744).
int tn_ranges(long M, long N, long K, int nz) {
  const long tiles = (M + kT - 1) / kT * ((N + kT - 1) / kT) * nz;
  if (tiles <= 0 || tiles > 128 || M * N * nz * 10 < tiles * kT * kT * 9) return 1;
  const long ks = 256 / tiles;
  return tiles * ks >= 224 && K >= 6144 * ks ? (int)ks : 1;
}
}  // namespace

size_t gemm_tn_parts_bytes(long M, long N, long K, int nz) {
  const int ks = tn_ranges(M, N, K, nz);
  return ks > 1 ? (size_t)ks * nz * M * ((N + 3) / 4 * 4) * 4 : 0;
}
int gemm_tn_ranges(const GemmArgs& g) {
  const size_t need = gemm_tn_parts_bytes(g.M, g.N, g.K, g.nz);
  return need && g.parts && need <= g.parts_bytes && gemm_tn_ok(g) ? tn_ranges(g.M, g.N, g.K, g.nz) : 1;
}
hipError_t launch_gemm_tn(const GemmArgs& g, hipStream_t s) { return g.M <= 0 || g.N <= 0 || g.nz <= 0 ? hipSuccess : launch_tn(g, 1, s); }
hipError_t launch_gemm_tn_ranges(const GemmArgs& g, hipStream_t s) {
  const int ks = gemm_tn_ranges(g);
  if (ks == 1) return launch_gemm_tn(g, s);
  const hipError_t e = launch_tn(g, ks, s);
  if (e != hipSuccess) return e;
  SumJob j = {};
  j.parts = g.parts; j.C = g.C; j.bias = g.bias; j.M = g.M; j.N = g.N; j.ksplit = ks; j.nz = g.nz;
  j.ldp = (g.N + 3) / 4 * 4; j.sPz = (long)ks * g.M * j.ldp; j.ldc = g.ldc; j.sCz = g.sCz; j.sbiasz = g.sbiasz; j.accumulate = g.accumulate;
  return finish_parts(j, gemm_tn_parts_bytes(g.M, g.N, g.K, g.nz), g.sums, s);
}

hipError_t launch_gemm_nt(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nz <= 0) return hipSuccess;
  NtArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K / 8 * 8; a.ktail = g.K % 8; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz;
  a.nseg = g.nseg; a.sAseg = g.sAseg; a.sBseg = g.sBseg; a.accumulate = g.accumulate;
  a.a_rows = g.a_rows; a.c_rows = g.c_rows; a.m_dev = g.m_dev; a.k_dev = g.k_dev; a.a_phys_rows = g.a_phys_rows; a.k_phys_rows = g.b_kcontig ? 0 : g.k_phys_rows;
  // the blocked raster pays when every XCD gets several blocks; with few tiles it would leave XCDs idle
  const int sups = cdiv(cdiv(g.M, kT), kSupM) * cdiv(cdiv(g.N, kT), kSupN);
  a.blocked = sups >= 32 ? 1 : 0;
  const int tiles = a.blocked ? cdiv(sups, 8) * 8 * kSupM * kSupN : cdiv(g.M, kT) * cdiv(g.N, kT);
  static std::atomic<unsigned long long> dl_attr_set{0};
  const hipError_t ea = once_per_device(dl_attr_set, [] {
    for (const void* k : {(const void*)gemm_dl8_f32_kernel<false>, (const void*)gemm_dl8_f32_kernel<true>,
                          (const void*)gemm_dl8_bf16_kernel<false>, (const void*)gemm_dl8_bf16_kernel<true>,
                          (const void*)gemm_nn8_f32_kernel<false>, (const void*)gemm_nn8_f32_kernel<true>}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kDlLds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
  if (ea != hipSuccess) return ea;
  const dim3 grid(tiles, g.nz);
  const bool ragged = a.K % kKB != 0, bf = g.out_bf16;
  if (!g.b_kcontig) {
    if (ragged || a.k_phys_rows % kKB != 0) hipLaunchKernelGGL(gemm_nn8_f32_kernel<true>, grid, dim3(512), kDlLds, s, a);
    else hipLaunchKernelGGL(gemm_nn8_f32_kernel<false>, grid, dim3(512), kDlLds, s, a);
  } else if (bf && ragged) hipLaunchKernelGGL(gemm_dl8_bf16_kernel<true>, grid, dim3(512), kDlLds, s, a);
  else if (bf) hipLaunchKernelGGL(gemm_dl8_bf16_kernel<false>, grid, dim3(512), kDlLds, s, a);
  else if (ragged) hipLaunchKernelGGL(gemm_dl8_f32_kernel<true>, grid, dim3(512), kDlLds, s, a);
  else hipLaunchKernelGGL(gemm_dl8_f32_kernel<false>, grid, dim3(512), kDlLds, s, a);
  return hipGetLastError();
}

hipError_t launch_frame_map(const int* lens, int T, int B, int* fidx, int* count, hipStream_t s) {
  if (T <= 0 || B <= 0) return hipSuccess;
  hipLaunchKernelGGL(frame_map_kernel, dim3(cdiv(T, 4)), dim3(256), 0, s, lens, T, B, fidx, count);
  return hipGetLastError();
}

hipError_t launch_pad_rows(const void* src, void* dst, long R, int C, int ld_dst, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  const long total = R * (ld_dst / 8);
  hipLaunchKernelGGL(pad_rows_kernel, dim3(cdiv(total, 256)), dim3(256), 0, s, (const uint16_t*)src, (uint4*)dst, R, C, ld_dst / 8);
  return hipGetLastError();
}

}  // namespace lstm
