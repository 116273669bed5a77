// bfloat16 products whose 256 x 256 tiles (gemm_nt.hip) would leave most of the device idle, and the layout those kernels lack:
//
//     C[M,N] (+)= sum_seg A_seg . B_seg (+ bias)     A, B each either k-contiguous or k-major:
//       NT  dX = DZ W_x^T                 both k-contiguous (a row per frame / per input feature)
//       NN  Zx = X W_x + b                A k-contiguous, B k-major: W_x as it lies in memory, no transposed copy
//       TN  dW_x = X^T DZ, dW_h           both k-major (a row per frame)
//
// What bounds these products in the large kernels is not the matrix cores: one sentence of 27 frames is 32 tiles of 256 x 256, each
// a walk over 32 stages of K at the latency of a load (1.6 us): 51 us for 0.9 GFLOP and 32 MB of weights, behind a transpose
// of those weights (17 us).  Here: tiles of 128 x 128, four wavefronts of 64 x 64 (2 x 2 MFMA blocks of 32 x 32 x 16), two work-groups per
// compute unit, and K cut into as many ranges as give the device 512 of them; the ranges' parts are added by a second kernel,
// which also applies bias, row map and rounding.
//
// Operands go from global memory straight into LDS (16 bytes per lane), K in stages of 64, two stages; the order within a stage
// and the reasons are those of gemm_nt.hip.  A k-contiguous operand sits there as rows of 128 bytes whose 16-byte slot p holds
// chunk p ^ ((row / 2) % 8); a k-major one as 64 rows of one k each whose 64-byte blocks are XORed with k % 4, read with the LDS
// transpose read.
//
// A stage is two phases of eight products: both operands k-contiguous, the first and the second row of blocks over all 64 k; else
// k-steps 0-1 and 2-3.  A phase's reads fetch the next one's fragments while its products run, a load behind each; what they have read is free
// when all wavefronts have met, once a phase, and is loaded again in the next one, so that half a stage to one and a half is always on its way.  A k-contiguous
// A with a k-major B goes out a whole stage at a time (its lines hold all 64 k, and W_x comes from memory: half a stage of 4000 columns at a time took 2 us of 30 more),
// B two stages ahead.  Before, a stage's loads went out together, a stage ahead, and were waited for together.  With the order of the tiles below, us, operands
// from memory: both k-contiguous 3200 x 2000 x 8000 135 and 127, 4096 x 2048 x 8192 158 and 140, 1120 x 2048 x 8192 114 and 79; k-major B
// 1120 x 8192 x 2048 69 and 56, 4096 x 2048 x 8192 178 and 144; both k-major 4096 x 2048 x 8192 163 and 148, 1000 x 8000 x 3200 70 and 68.  What bounds them now
// is the path from L2 to LDS: of 138 us without the products 120 remain, without the loads 108 (1270 TFLOP/s).  Tried without gain: a phase
// a quarter of a stage (130, 137 and 74 us of the first three), ten quarters of a stage in 80 KiB of LDS (128, 143, 80), three or four whole stages with one
// work-group per compute unit.
#include "gemm_plan.h"
#include "recurrent_dev.h"
#include <algorithm>
#include <type_traits>

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices
constexpr unsigned kParked = 0x7ffffff0u;
constexpr int kKB = kTileK;             // k per stage

struct TileArgs {
  const char* A; const char* B; void* C; const float* bias;
  int M, N, K;
  int ktail;                              // both operands k-contiguous: four k behind the K (a multiple of 8) that the stages walk
  long lda, ldb, ldc;                     // elements
  long sAz, sBz, sCz, sbiasz; int nz;
  int nseg; long sAseg, sBseg;
  int accumulate;
  const int* a_rows; const int* c_rows; int a_phys_rows;   // (see GemmArgs)
  const int* k_rows; int k_phys_rows;     // NN without k_rows: k_phys_rows > 0 is the number of rows B has (fewer than K: A's padding)
  const int* m_dev; const int* k_dev;
  int ksplit; float* parts; long ldp;     // > 1: range r of problem z stores its part at parts[(z * ksplit + r) * M * ldp ..], rows packed
};

struct TileGroup { TileArgs p[2]; int first1; };         // blocks from first1 on are the second product's
struct TileTrio { TileArgs p[3]; int first1, first2; };

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
__device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kTM = kTileEdge, kTN = kTileEdge;
constexpr int kOpBytes = 128 * kKB * 2, kStageBytes = 2 * kOpBytes;                  // one operand of a stage, both
constexpr int kEpStride = kTN + 4, kEpBytes = 64 * kEpStride * 4;                    // the epilogue stages 64 rows at a time
constexpr int tile_lds(bool ak, bool bk) { return 2 * kStageBytes + (ak && !bk ? kOpBytes : 0); }      // (k-contiguous A, k-major B: a third stage of B)
static_assert(2 * kStageBytes >= kEpBytes && 2 * tile_lds(true, false) <= 160 * 1024, "two work-groups to a compute unit");

// KROWS: k-major operands whose row k is row k_rows[k] in memory.  PACED (both k-contiguous): half as much on its way (see paced()).
template <typename TC, bool AK, bool BK, bool KROWS, bool PACED>
__device__ __forceinline__ void tile_body(const TileArgs& g, int mine, char* lds) {       // mine: work-group of this product
  constexpr int NW = 4;
  constexpr bool kMixed = AK && !BK;
  constexpr bool kHalves = AK && BK;      // a phase is one row of blocks, half of them, over the stage's 64 k (else: all blocks over 32 k)
  static_assert(!KROWS || (!AK && !BK), "a list of rows: both operands k-major");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int r = lane & 31, gq = lane >> 5;

  // Work-groups are dealt to the 8 XCDs round-robin.  Up to as many tile rows as columns: bands of 8 tile columns, row-major inside a band, so
  // that each XCD keeps one tile column of B in its L2 and neighbouring columns are read and written at the same time.  More rows: each XCD would
  // read all of A, and takes an eighth of all tiles instead, one behind the other in an order of bands of `high` rows, about as many rows as columns at a
  // time (us, bands of columns and these: 4096 x 2048 x 8192 157 and 139, 3200 x 2000 x 8000 141 and 130; but 1120 x 8192 x 2048 with k-major B 55 and 57).
  // Not for K ranges of up to five stages, which are over before neighbours drift apart (a layer's forward pass, n = 136, both directions, us: n_in = 620, five stages,
  // 1600 frames 72 and 75, 1280 frames 69 and 70; n_in = 2000, 1600 frames, eight stages 79 and 75, 960 frames, a little more than five, 72 and 71).
  // Both operands k-major, several K ranges or directions: no two of them read the same rows, so always an eighth each, whole ranges where they come out even; dealt
  // round, every XCD read every row of A (both products of weight gradients, us, a round / an eighth: 24955 frames, both directions, n = 296, n_in = 592
  // 221 / 153, n_in = 65 124 / 79; 9600 frames of n = 200, n_in = 400 66 / 42; 16000 of n = 512, n_in = 1024 222 / 220).
  const int M = g.m_dev ? min(g.M, *g.m_dev) : g.M, K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  const int ktiles = (K + kKB - 1) / kKB;
  const int tiles_m = (M + kTM - 1) / kTM, tiles_n = (g.N + kTN - 1) / kTN, per_z = tiles_m * tiles_n, tiles = per_z * g.nz * g.ksplit;
  const int each = (tiles + 7) >> 3;
  const bool apart = !AK && !BK && g.nz * g.ksplit > 1;
  const bool by_rows = apart || (tiles_m > tiles_n && (g.ksplit == 1 || ktiles * g.nseg > 5 * g.ksplit));
  // B k-major, bands of columns, some units with two work-groups: an eighth of all tiles each as well, where a tile column is not one XCD's.  In whole eights of columns it is, and stays
  // in that L2; else an XCD's column changes from row to row of the last band, and with loads a stage and a half ahead such products had become slower than before them (us, before those
  // loads / a round / an eighth): both k-major 640 x 9000 x 3200 67 / 71 / 57, 1576 x 3704 x 6288 125 / 135 / 126, 408 x 9784 x 5000 103 / 109 / 89; A k-contiguous, the last, 101 / 108 / 100.  A round where
  // it is no slower: whole eights (1280 x 4096 x 6288, both k-major, 89 / 99), fewer work-groups (1920 x 2280 x 2048, 270, 35.8 / 37.6) or more (608 x 11856 x 2584, both k-major, 465, 63 / 67), three
  // rows of tiles (384 x 18000 x 1024 31.8 / 32.8), a short K (1376 x 4240 x 536 20.6 / 21.3).
  const bool wanders = !BK && g.nz * g.ksplit == 1 && tiles_m >= 4 && tiles_m <= tiles_n && tiles_n % 8 != 0 && tiles >= 300 && tiles < 440 && ktiles >= 16;
  const bool eighths = by_rows || wanders;
  const int idx = eighths ? (mine & 7) * each + (mine >> 3) : mine;
  if (idx >= tiles || (eighths && (mine >> 3) >= each)) return;
  const int zk = idx / per_z, bid = idx - zk * per_z;
  int tm, tn;
  if (by_rows) {
    int side = 1;
    while (side < 8 && (side + 1) * (side + 1) <= each) ++side;
    const int bands = max(1, (tiles_m + side / 2) / side), high = (tiles_m + bands - 1) / bands;
    const int band = bid / (high * tiles_n), height = min(high, tiles_m - band * high), rel = bid - band * high * tiles_n;
    tm = band * high + rel % height; tn = rel / height;
  } else {
    const int band = bid / (8 * tiles_m), width = min(8, tiles_n - band * 8), rel = bid - band * 8 * tiles_m;
    tm = rel / width; tn = band * 8 + rel % width;
  }
  const int m0 = __builtin_amdgcn_readfirstlane(tm * kTM), n0 = __builtin_amdgcn_readfirstlane(tn * kTN);
  const int ksplit = g.ksplit, z = __builtin_amdgcn_readfirstlane(zk / ksplit), ks = __builtin_amdgcn_readfirstlane(zk - z * ksplit);

  const int nstage = ktiles * g.nseg;
  const int tail_chunks = (K - (ktiles - 1) * kKB + 7) >> 3;   // 16-byte chunks of a k-contiguous operand in the last k-tile
  // (told to be wave-uniform: divisions leave them in vector registers)
  const int it0 = __builtin_amdgcn_readfirstlane(nstage * ks / ksplit), total = __builtin_amdgcn_readfirstlane(nstage * (ks + 1) / ksplit) - it0;

  // Loads.  k-contiguous operand, half h (rows of every wavefront's first or second block), load j: rows 64 j + 32 h + 8 wave .. + 7,
  // lane l slot l & 7 of row l >> 3.  k-major operand, k-step s: k-rows 16 s + 4 wave .. + 3, lane l slot l % 16 of row l / 16.
  const int kk = lane >> 4;                                    // k-major: this lane's row of a load's four
  const int kc_chunk = (lane & 7) ^ ((((wave & 1) * 8 + (lane >> 3)) >> 1) & 7), km_chunk = (lane & 15) ^ (4 * kk);
  const bool past = kc_chunk >= tail_chunks;                   // k-contiguous: this lane's chunk lies past a ragged last k-tile
  const unsigned lda2 = (unsigned)g.lda * 2u, ldb2 = (unsigned)g.ldb * 2u;
  const auto clip = [](long o, bool ok) { return ok && o <= 0x7ffffe00L ? (unsigned)o : kParked; };
  unsigned va[AK ? 4 : 1], vb[BK ? 4 : 1];                     // k-contiguous: [2 h + j]
  if constexpr (AK) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = m0 + (q & 1) * 64 + (q >> 1) * 32 + wave * 8 + (lane >> 3);
      const long pr = row < M ? (g.a_rows ? (long)g.a_rows[row] : row) : -1;
      va[q] = clip(pr * g.lda * 2 + kc_chunk * 16, pr >= 0);
    }
  } else {
    va[0] = clip((KROWS ? 0L : (wave * 4 + kk) * g.lda * 2) + ((long)m0 + km_chunk * 8) * 2, m0 + km_chunk * 8 < M);
  }
  if constexpr (BK) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = n0 + (q & 1) * 64 + (q >> 1) * 32 + wave * 8 + (lane >> 3);
      vb[q] = clip((long)row * g.ldb * 2 + kc_chunk * 16, row < g.N);
    }
  } else {
    vb[0] = clip((KROWS ? 0L : (wave * 4 + kk) * g.ldb * 2) + ((long)n0 + km_chunk * 8) * 2, n0 + km_chunk * 8 < g.N);
  }
  const int KB = AK && !BK && g.k_phys_rows > 0 ? g.k_phys_rows : K;
  const long k_mem = KROWS ? g.k_phys_rows : KB;
  const auto rec_of = [](long b) { return (unsigned)(b > 0x7fffff00L ? 0x7fffff00L : b); };
  const unsigned a_rec = rec_of((AK ? (long)(g.a_rows ? g.a_phys_rows : M) : k_mem) * g.lda * 2), b_rec = rec_of((BK ? (long)g.N : k_mem) * g.ldb * 2);
  const char* const a_base = g.A + g.sAz * z * 2;
  const char* const b_base = g.B + g.sBz * z * 2;
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;

  struct Stage { int it, seg, kt; };                           // the stage whose loads go out: place in this range, segment, k-tile inside it
  const int seg0 = g.nseg > 1 ? __builtin_amdgcn_readfirstlane(it0 / ktiles) : 0;
  Stage nx = {0, seg0, it0 - seg0 * ktiles};
  Stage nb = nx;                                               // kMixed: of B
  auto advance = [&](Stage& t) __attribute__((always_inline)) {
    ++t.it;
    if (++t.kt == ktiles && kHalves) { t.kt = 0; ++t.seg; }
  };
  int b_out = 0, b_in = 0;                                     // kMixed: stage it of B is the (it % 3)th
  auto next = [&](int& slot) __attribute__((always_inline)) { slot = slot == 2 * kOpBytes ? 0 : slot + kOpBytes; };
  // where stage `it` of an operand lies (`slot`: of a kMixed B)
  auto place = [&](bool is_a, int it, int slot) __attribute__((always_inline)) {
    if constexpr (kMixed) return is_a ? (it & 1) * kOpBytes : 2 * kOpBytes + slot;
    return (it & 1) * kStageBytes + (is_a ? 0 : kOpBytes);
  };
  // (past the last stage the same loads are issued with every lane outside the descriptor: the counted waits below count them)
  auto issue_half = [&](bool is_a, int h, int j) __attribute__((always_inline)) {
    const u32x4 rs = is_a ? make_rsrc(a_base + (long)g.sAseg * nx.seg * 2, nx.it < total ? a_rec : 0u) : make_rsrc(b_base + (long)g.sBseg * nx.seg * 2, nx.it < total ? b_rec : 0u);
    const unsigned dst = lds_base + place(is_a, nx.it, 0) + (h * 32 + wave * 8) * 128;
    const bool cut = past && nx.kt == ktiles - 1;
    load_to_lds_b128(rs, dst + j * 64 * 128, cut ? kParked : is_a ? va[AK ? 2 * h + j : 0] : vb[BK ? 2 * h + j : 0], (unsigned)nx.kt * (kKB * 2));
  };
  // With KROWS the memory rows are entries of the packed list, looked up a phase ahead by scalar loads that are waited for together with
  // the operand loads (see gemm_nt.hip).  The list is readable up to the next multiple of 64 entries.
  i32x4 prow[8];
  auto lookup = [&](int dst, int kt, int s) __attribute__((always_inline)) {
    if constexpr (KROWS) {
      const int* p = g.k_rows + (long)min(kt, ktiles - 1) * kKB + s * 16 + wave * 4;
      asm volatile("s_load_dwordx4 %0, %1, 0x0" : "=s"(prow[dst]) : "s"(p) : "memory");
    }
  };
  const unsigned odd = (kk & 1) ? ~0u : 0u, upper = (kk & 2) ? ~0u : 0u;                 // which of a load's four entries is this lane's
  auto issue_rows = [&](bool is_a, int s, int entry) __attribute__((always_inline)) {    // k-step s of a k-major operand
    const Stage& t = kMixed ? nb : nx;
    const u32x4 rs = make_rsrc(is_a ? a_base : b_base, t.it < total ? (is_a ? a_rec : b_rec) : 0u);
    const unsigned ld2 = is_a ? lda2 : ldb2;
    unsigned v = is_a ? va[0] : vb[0];
    if constexpr (KROWS) {                                     // (32-bit arithmetic: the operands end below 2^31; a parked column stays past the end)
      const i32x4 p4 = prow[entry];
      const unsigned lo = ((unsigned)p4[0] & ~odd) | ((unsigned)p4[1] & odd), hi = ((unsigned)p4[2] & ~odd) | ((unsigned)p4[3] & odd);
      v = ((lo & ~upper) | (hi & upper)) * ld2 + v;
    }
    if (s * 16 + wave * 4 + kk >= KB - t.kt * kKB) v = kParked;
    load_to_lds_b128(rs, lds_base + place(is_a, t.it, b_out) + (s * NW + wave) * 1024, v, KROWS ? 0u : (unsigned)(t.kt * kKB + s * 16) * ld2);
  };

  // Fragments of k-step s (16 k): k-contiguous: row r of a block, chunk 2 s + gq; k-major: two transpose reads (see gemm_nt.hip).
  const int kc_off = r * 128 + ((gq ^ ((r >> 1) & 7)) * 16);
  const int l16 = lane & 15, sw = (l16 >> 2) & 3;
  const int km_row = gq * 8 + (l16 >> 2), km_low = ((lane >> 4) & 1) * 32 + (l16 & 3) * 8;
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  auto tr_read = [&](const char* p) __attribute__((always_inline)) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * 256));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    return make_uint4(l2.x, l2.y, h2.x, h2.y);
  };
  // block i of this wavefront's two, k-step s
  auto frag = [&](bool is_a, int it, int i, int s) __attribute__((always_inline)) {
    const char* base = lds + place(is_a, it, b_in);
    const int blk = (is_a ? wm : wn) * 2 + i;
    if (is_a ? AK : BK) return *(const uint4*)(base + blk * 32 * 128 + (kc_off ^ (s * 32)));
    return tr_read(base + (s * 16 + km_row) * 256 + (((blk ^ sw) & 3) << 6) + km_low);
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  if (kHalves && g.ktail && ks == 0) {
    for (int seg = 0; seg < g.nseg; ++seg) {
      uint2 ta[2], tb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int ra = m0 + (wm * 2 + i) * 32 + r, rb = n0 + (wn * 2 + i) * 32 + r;
        ta[i] = tb[i] = make_uint2(0u, 0u);
        if (gq == 0 && ra < M) ta[i] = *(const uint2*)(a_base + (g.sAseg * seg + (long)(g.a_rows ? g.a_rows[ra] : ra) * g.lda + K) * 2);
        if (gq == 0 && rb < g.N) tb[i] = *(const uint2*)(b_base + (g.sBseg * seg + (long)rb * g.ldb + K) * 2);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q >> 1][q & 1] = mma_last4(ta[q >> 1], tb[q & 1], acc[q >> 1][q & 1]);
    }
  }
  // The end of a phase: this wavefront's reads have returned (what they read may be overwritten once all have met), and what the phase
  // after next multiplies has landed (`younger` loads went out behind it).
  auto end_phase = [&](auto younger) __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070 | decltype(younger)::value);
    if constexpr (KROWS) asm volatile("" : "+s"(prow[0]), "+s"(prow[1]), "+s"(prow[2]), "+s"(prow[3])::"memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  const auto c4 = std::integral_constant<int, 4>{};
  const auto c8 = std::integral_constant<int, 8>{};
  const auto c10 = std::integral_constant<int, 10>{};
  const auto c12 = std::integral_constant<int, 12>{};

  // One stage or two: nothing to overlap, so all loads and then all products.  The pipeline's loads past the end, its barriers and its last wait cost as
  // much as the work (us, pipeline / this; k-major B: 3200 x 2000 x 40 10.2 / 9.4, x 128 11.1 / 10.2, 5000 x 2048 x 64 17.0 / 15.8; both k-contiguous: 3200 x 2000 x 64
  // 10.0 / 9.4, x 128 10.6 / 10.2).
  if (!KROWS && total <= 2) {
    for (int k = 0; k < total; ++k) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (AK) issue_half(true, q >> 1, q & 1); else issue_rows(true, q, 0);
        if constexpr (BK) issue_half(false, q >> 1, q & 1); else issue_rows(false, q, 0);
      }
      if constexpr (kMixed) { advance(nb); next(b_out); }
      advance(nx);
    }
    end_phase(std::integral_constant<int, 0>{});
    for (int it = 0; it < total; ++it) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint4 a[2] = {frag(true, it, 0, s), frag(true, it, 1, s)}, b[2] = {frag(false, it, 0, s), frag(false, it, 1, s)};
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q >> 1][q & 1] = mma(a[q >> 1], b[q & 1], acc[q >> 1][q & 1]);
      }
      if constexpr (kMixed) next(b_in);
    }
  } else if constexpr (kHalves) {
    uint4 fa[2][4], fb[2][2][4];
    // the products of row i, a load behind each: f(number of the product)
    auto mul = [&](int i, const uint4 (&y)[2][4], auto&& f) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        acc[i][m & 1] = mma(fa[i][m >> 1], y[m & 1][m >> 1], acc[i][m & 1]);
        __builtin_amdgcn_sched_barrier(0);
        f(m);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto read = [&](uint4 (&f)[4], bool is_a, int it, int i) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 4; ++s) f[s] = frag(is_a, it, i, s);
    };
    auto stage = [&](int it, auto parity) __attribute__((always_inline)) {
      constexpr int par = decltype(parity)::value;
      const auto pace = std::integral_constant<int, PACED ? 4 : 8>{};
      read(fa[1], true, it, 1);
      mul(0, fb[par], [&](int m) __attribute__((always_inline)) { if (m < 6) issue_half(m < 2, m >> 2, m & 1); });
      end_phase(pace);
      read(fa[0], true, it + 1, 0);
      read(fb[par ^ 1][0], false, it + 1, 0);
      read(fb[par ^ 1][1], false, it + 1, 1);
      mul(1, fb[par], [&](int m) __attribute__((always_inline)) {
        if (m < 2) issue_half(true, 1, m);
        if (m == 2) advance(nx);
      });
      end_phase(pace);
    };
    if (total > 0) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int q = 0; q < 8; ++q) issue_half(q < 2 || q > 5, q >> 2, q & 1);
        advance(nx);
      }
      end_phase(c10);
      read(fa[0], true, 0, 0);
      read(fb[0][0], false, 0, 0);
      read(fb[0][1], false, 0, 1);
      end_phase(c8);
      for (int it = 0; it < total; it += 2) {
        stage(it, std::integral_constant<int, 0>{});
        if (it + 1 < total) stage(it + 1, std::integral_constant<int, 1>{});
      }
    }
  } else {
    uint4 fa[2][2][2], fb[2][2][2];                            // [half of a stage][k-step][block]
    auto read = [&](int it, int h) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          fa[h][s][i] = frag(true, it, i, 2 * h + s);
          fb[h][s][i] = frag(false, it, i, 2 * h + s);
        }
      if (kMixed && h == 1) next(b_in);
    };
    // What goes out in half h: its k-steps of stage nx; with a k-contiguous A nothing in the first half, all of A's and B's stages in the second.
    auto issue = [&](int h, int m, int entry) __attribute__((always_inline)) {         // the load behind product m of a phase
      if constexpr (AK) {
        if (h == 1 && m < 4) issue_half(true, m >> 1, m & 1);
        if (h == 1 && m >= 4) issue_rows(false, m - 4, entry);
        if (h == 1 && m == 7) { advance(nb); next(b_out); }
      } else if (m < 4) {
        issue_rows(m < 2, 2 * h + (m & 1), entry + (m & 1));
      }
      if (h == 1 && m == 7) advance(nx);
    };
    auto phase = [&](int it, int h, auto younger) __attribute__((always_inline)) {
      // (first: a look-up that misses the scalar cache takes most of a phase)
      lookup(2 * (h ^ 1), nx.kt + h, 2 * (h ^ 1));
      lookup(2 * (h ^ 1) + 1, nx.kt + h, 2 * (h ^ 1) + 1);
      read(it + h, h ^ 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        acc[(m >> 1) & 1][m & 1] = mma(fa[h][m >> 2][(m >> 1) & 1], fb[h][m >> 2][m & 1], acc[(m >> 1) & 1][m & 1]);
        __builtin_amdgcn_sched_barrier(0);
        issue(h, m, 2 * h);
        __builtin_amdgcn_sched_barrier(0);
      }
      end_phase(younger);
    };
    if (total > 0) {
      if constexpr (KROWS) {
#pragma unroll
        for (int k = 0; k < 8; ++k) lookup(k, nx.kt + (k >> 2), k & 3);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(prow[0]), "+s"(prow[1]), "+s"(prow[2]), "+s"(prow[3]), "+s"(prow[4]), "+s"(prow[5]), "+s"(prow[6]), "+s"(prow[7])::"memory");
      }
#pragma unroll
      for (int k = 0; k < 32; ++k) {
        if (kMixed && k == 8) {                                // B's first stage, then A's with B's next
#pragma unroll
          for (int s = 0; s < 4; ++s) issue_rows(false, s, 0);
          advance(nb); next(b_out);
        }
        issue((k >> 3) & 1, k & 7, k >> 3 << 1);
      }
      lookup(0, nx.kt, 0);
      lookup(1, nx.kt, 1);
      end_phase(c12);
      read(0, 0);
      if constexpr (AK) end_phase(c12); else end_phase(c8);
      for (int it = 0; it < total; ++it) {
        if constexpr (AK) {
          phase(it, 0, c4); phase(it, 1, c12);
        } else {
          phase(it, 0, c8); phase(it, 1, c8);
        }
      }
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070);                          // vmcnt(0) lgkmcnt(0): the epilogue uses LDS

  // Epilogue: 32 rows of every wavefront row at a time through LDS, out as whole rows.
  constexpr int kTpr = kTN / 4;                                 // threads per row
  const bool to_parts = ksplit > 1;
  TC* C = (TC*)g.C + g.sCz * z;
  float* P = g.parts + (long)(z * ksplit + ks) * g.M * g.ldp;
  const float* bias = g.bias && !to_parts ? g.bias + g.sbiasz * z : nullptr;
  float* ep = (float*)lds;
  const int col = n0 + (tid % kTpr) * 4;
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if (bias) {
#pragma unroll
    for (int k = 0; k < 4; ++k) if (col + k < g.N) bv[k] = bias[col + k];
  }
  const bool whole = col + 3 < g.N, vec = whole && g.ldc % 4 == 0 && g.sCz % 4 == 0 && ((uintptr_t)g.C & 15u) == 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) ep[(wm * 32 + 8 * (v >> 2) + 4 * gq + (v & 3)) * kEpStride + (wn * 2 + j) * 32 + r] = acc[i][j][v];
    __syncthreads();
    if (col < g.N) {
      constexpr int kStep = 64 * NW / kTpr, kIts = 64 / kStep;
      int crow[kIts];                                          // (looked up before the first store: a load behind a store waits for it)
#pragma unroll
      for (int q = 0; q < kIts; ++q) {
        const int rl = tid / kTpr + q * kStep, row = min(m0 + (rl >> 5) * 64 + i * 32 + (rl & 31), M - 1);
        crow[q] = g.c_rows && !to_parts ? g.c_rows[row] : row;
      }
#pragma unroll
      for (int q = 0; q < kIts; ++q) {
        const int rl = tid / kTpr + q * kStep, row = m0 + (rl >> 5) * 64 + i * 32 + (rl & 31);
        if (row >= M) continue;
        const float4 val = *(const float4*)&ep[rl * kEpStride + (tid % kTpr) * 4];
        if (to_parts) {                                        // (ldp is a multiple of 4; what lies past N is padding)
          *(float4*)(P + (long)row * g.ldp + col) = val;
          continue;
        }
        float e[4] = {val.x + bv[0], val.y + bv[1], val.z + bv[2], val.w + bv[3]};
        const long off = (long)crow[q] * g.ldc + col;
        if constexpr (sizeof(TC) == 4) {
          float* Cf = (float*)C + off;
          if (vec && !g.accumulate) __builtin_nontemporal_store((f32x4){e[0], e[1], e[2], e[3]}, (f32x4*)Cf);
          else if (vec) {
            const float4 o = *(const float4*)Cf;
            *(float4*)Cf = make_float4(e[0] + o.x, e[1] + o.y, e[2] + o.z, e[3] + o.w);
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) if (col + k < g.N) Cf[k] = g.accumulate ? Cf[k] + e[k] : e[k];
          }
        } else {
          uint16_t* Cb = (uint16_t*)C + off;
          if (vec) *(uint2*)Cb = make_uint2(f2bf_bits(e[0]) | ((unsigned)f2bf_bits(e[1]) << 16), f2bf_bits(e[2]) | ((unsigned)f2bf_bits(e[3]) << 16));
          else {
#pragma unroll
            for (int k = 0; k < 4; ++k) if (col + k < g.N) Cb[k] = f2bf_bits(e[k]);
          }
        }
      }
    }
  }
}

template <typename TC, bool AK, bool BK, bool KROWS, bool PACED>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(TileGroup grp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const bool second = (int)blockIdx.x >= grp.first1;
  const TileArgs g = second ? grp.p[1] : grp.p[0];
  tile_body<TC, AK, BK, KROWS, PACED>(g, (int)blockIdx.x - (second ? grp.first1 : 0), lds);
}
// The three products of a layer's backward pass: dX, both operands k-contiguous, then dW_x and dW_h, both k-major.
template <typename TC, bool KROWS>
__global__ __launch_bounds__(256, 2) void gemm_tile_grads_kernel(TileTrio grp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if ((int)blockIdx.x < grp.first1) {
    const TileArgs g = grp.p[0];
    tile_body<TC, true, true, false, false>(g, blockIdx.x, lds);
  } else {
    const bool last = (int)blockIdx.x >= grp.first2;
    const TileArgs g = last ? grp.p[2] : grp.p[1];
    tile_body<float, false, false, KROWS, false>(g, (int)blockIdx.x - (last ? grp.first2 : grp.first1), lds);
  }
}

int blocks_of(const TileArgs& a) { return (cdiv(a.M, kTM) * cdiv(a.N, kTN) * a.nz * a.ksplit + 7) / 8 * 8; }
template <typename TC, bool KROWS>
hipError_t launch_grads_as(TileTrio a, hipStream_t s) {
  const auto kernel = gemm_tile_grads_kernel<TC, KROWS>;
  constexpr int lds = std::max(tile_lds(true, true), tile_lds(false, false));
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [&] { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (ea != hipSuccess) return ea;
  a.first1 = blocks_of(a.p[0]);
  a.first2 = a.first1 + blocks_of(a.p[1]);
  hipLaunchKernelGGL(kernel, dim3(a.first2 + blocks_of(a.p[2])), dim3(256), lds, s, a);
  return hipGetLastError();
}
template <typename TC, bool AK, bool BK, bool KROWS, bool PACED = false>
hipError_t launch_as(const TileGroup& a, int count, hipStream_t s) {
  const auto kernel = gemm_tile_kernel<TC, AK, BK, KROWS, PACED>;
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [&] { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds(AK, BK)); });
  if (ea != hipSuccess) return ea;
  TileGroup c = a;
  int blocks[2] = {0, 0};
  for (int i = 0; i < count; ++i) blocks[i] = blocks_of(c.p[i]);
  c.first1 = count == 2 ? blocks[0] : 0x7fffffff;
  hipLaunchKernelGGL(kernel, dim3(blocks[0] + blocks[1]), dim3(256), tile_lds(AK, BK), s, c);
  return hipGetLastError();
}
// Up to 256 work-groups have a compute unit each, from 512 on they share it two by two.  In between those alone run ahead of those that share, whose operands
// have left L2 by the time that they ask for them.  With half as much on its way (a wait for 4 younger loads instead of 8) those alone are slower and the
// launch ends earlier (work-groups; us, 8 / 4, operands from memory): 1408 x 4000 x 4000 (352) 81 / 76, 1600 x 4000 x 4000 (416) 77 / 72, 1920 x 4000 x 8000
// (480) 138 / 125, 384 x 20000 x 1024 (471) 28 / 26; but 1280 x 4000 x 8000 (320) 109 / 111, 2400 x 4000 x 2048 (608) 51 / 60.  In the order by rows neighbours share
// more of what they read, and less on its way is no gain: 6656 x 1000 x 2048 (416) 37 / 41.
// They run ahead the further the longer K is, and A, which the rows of tiles share, the sooner the fewer rows there are.  On a shorter K less on its way is a loss: 1576 x 4696 (13 rows of
// tiles) x 512 20.4 / 21.6, x 1536 33.4 / 35.0, x 2048 44.0 / 43.5; 2000 x 3000 (16) x 1024 23.5 / 24.8, x 2048 36.3 / 36.2; 900 x 8000 (8) x 768 21.0 / 21.2, x 1280 34.7 / 30.2;
// 640 x 11000 (5) x 512 18.8 / 20.0, x 1024 30.1 / 28.0; 384 x 20000 (3) x 256 14.1 / 14.3, x 512 20.6 / 18.6.
bool paced(const TileArgs& a) {
  const long tiles_m = cdiv(a.M, kTM), tiles_n = cdiv(a.N, kTN), groups = tiles_m * tiles_n * a.nz * a.ksplit;
  return tiles_m <= tiles_n && groups >= 352 && groups < 512 && (long)a.K * a.nseg / a.ksplit >= std::min(160 * tiles_m, 2048L);
}
template <typename TC>
hipError_t launch_layout(const TileGroup& a, int count, bool ak, bool bk, hipStream_t s) {
  if (ak && bk) return paced(a.p[0]) ? launch_as<TC, true, true, false, true>(a, count, s) : launch_as<TC, true, true, false>(a, count, s);
  if (ak) return launch_as<TC, true, false, false>(a, count, s);
  if (a.p[0].k_rows) return launch_as<TC, false, false, true>(a, count, s);
  return launch_as<TC, false, false, false>(a, count, s);
}

TileProduct sizes_of(const GemmArgs& g) { return {g.M, g.N, g.K, g.nz, g.nseg}; }
long tiles_of(const GemmArgs& g) { return tile_count(g.M, g.N, g.nz); }
int ranges_of(const GemmArgs& g, long others) { return tile_ranges(tiles_of(g), others, tile_stages(g.K, g.nseg)); }
TileArgs tile_args(const GemmArgs& g, int ks, size_t parts_used) {
  TileArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  const bool halves = g.a_kcontig && g.b_kcontig;
  a.M = g.M; a.N = g.N; a.K = halves ? g.K / 8 * 8 : g.K; a.ktail = halves ? g.K % 8 : 0; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz;
  a.nseg = g.nseg; a.sAseg = g.sAseg; a.sBseg = g.sBseg; a.accumulate = g.accumulate;
  a.a_rows = g.a_rows; a.c_rows = g.c_rows; a.a_phys_rows = g.a_phys_rows; a.k_rows = g.k_rows; a.k_phys_rows = g.k_phys_rows;
  a.m_dev = g.m_dev; a.k_dev = g.k_dev;
  a.ldp = (g.N + 3) / 4 * 4;
  a.ksplit = g.parts ? ks : 1;
  if (parts_used + tile_part_bytes(g.M, g.N, g.nz, a.ksplit) > g.parts_bytes) a.ksplit = 1;
  a.parts = a.ksplit > 1 ? (float*)((char*)g.parts + parts_used) : nullptr;
  return a;
}
hipError_t finish(const TileArgs& a, const GemmArgs& g, hipStream_t s) {
  if (a.ksplit == 1) return hipGetLastError();
  SumJob j = {};
  j.parts = a.parts; j.C = a.C; j.bias = a.bias; j.M = a.M; j.N = a.N; j.ksplit = a.ksplit; j.nz = a.nz;
  j.ldp = a.ldp; j.sPz = (long)a.ksplit * a.M * a.ldp; j.ldc = a.ldc; j.sCz = a.sCz; j.sbiasz = a.sbiasz;
  j.c_rows = a.c_rows; j.m_dev = a.m_dev; j.accumulate = a.accumulate; j.out_bf16 = g.out_bf16;
  return finish_parts(j, tile_part_bytes(a.M, a.N, a.nz, a.ksplit), g.sums, s);
}

}  // namespace

bool gemm_tile_ok(const GemmArgs& g) {
  const auto a8 = [](const void* p) { return ((uintptr_t)p & 7u) == 0; };       // (see gemm_nt_ok)
  const long lim = 0x7ffffe00L;           // operands are addressed with 32-bit byte offsets
  const long k_rows = g.k_phys_rows > 0 ? g.k_phys_rows : g.K, a_rows = g.a_kcontig ? (g.a_rows ? g.a_phys_rows : g.M) : k_rows;
  if (a_rows * g.lda * 2 > lim || (g.b_kcontig ? (long)g.N : k_rows) * g.ldb * 2 > lim) return false;
  if (g.a_kcontig && (g.K % (g.b_kcontig ? 4 : 8) != 0 || g.K < 8 || (g.k_dev && g.K % 64 != 0))) return false;   // whole chunks, or a half at the end of both; a device-resident K counts whole stages there
  if (!g.a_kcontig && (g.b_kcontig || g.a_rows || g.m_dev || g.nseg > 1)) return false;
  if (g.a_kcontig && !g.b_kcontig && (g.k_rows || g.nseg > 1)) return false;
  return g.in_bf16 && !g.lens && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.sAz % 4 == 0 && g.sBz % 4 == 0 && g.sAseg % 4 == 0 && g.sBseg % 4 == 0 &&
         a8(g.A) && a8(g.B) && !(g.accumulate && g.out_bf16);
}

// Fewer 256 x 256 tiles than fill the device's 256 compute units: those of gemm_nt.hip would leave some idle for the whole product.  us there / here, all rows real,
// operands from memory: both k-contiguous 3000 x 2300 x 2048 (108 tiles) 46 / 38, 3300 x 2800 x 2048 (143) 47 / 53, 3300 x 4000 x 2048 (208) 56 / 74; k-major B, 143
// tiles, 46 / 58; both k-major, 3000 x 3600 x 1000 (180) 35 / 38, 3296 x 4000 x 1000 (208) 37 / 46.  The count is of padded rows, though, and a batch of sequences is often half
// padding: 200 tiles then hold 100 real ones, which is where the two are equal (1600 real of 3000 rows x 4000 x 1000, 192 tiles: 55 / 24).
bool gemm_tile_small(long M, long N, int nz) { return (long)cdiv(M, 256) * cdiv(N, 256) * nz <= 200; }

size_t gemm_tile_parts_bytes(long M, long N, long K, int nz, int nseg) {
  return tile_part_bytes(M, N, nz, tile_ranges(tile_count(M, N, nz), 0, tile_stages(K, nseg)));
}

hipError_t launch_gemm_tile(const GemmArgs& g, hipStream_t s) {
  TileGroup a = {};
  a.p[0] = tile_args(g, ranges_of(g, 0), 0);
  const bool bf = g.out_bf16 && a.p[0].ksplit == 1;
  const hipError_t e = bf ? launch_layout<uint16_t>(a, 1, g.a_kcontig, g.b_kcontig, s) : launch_layout<float>(a, 1, g.a_kcontig, g.b_kcontig, s);
  return e == hipSuccess ? finish(a.p[0], g, s) : e;
}

// dW_x and dW_h: each alone leaves the device's last work-groups waiting for it, and wants twice the K ranges to fill the device.
hipError_t launch_gemm_tile_pair(const GemmArgs& g, const GemmArgs& h, hipStream_t s) {
  if (g.M <= 0 || h.M <= 0 || g.N <= 0 || h.N <= 0 || g.nz <= 0) return hipErrorInvalidValue;
  TileGroup a = {};
  a.p[0] = tile_args(g, ranges_of(g, tiles_of(h)), 0);
  a.p[1] = tile_args(h, ranges_of(h, tiles_of(g)), tile_part_room(g.M, g.N, g.nz, a.p[0].ksplit));
  hipError_t e = launch_layout<float>(a, 2, false, false, s);
  if (e != hipSuccess || (e = finish(a.p[0], g, s)) != hipSuccess) return e;
  return finish(a.p[1], h, s);
}

// dX needs dZ and W_x, dW_x and dW_h need dZ, x and h: none waits for another, and each alone ends with most of the device idle (us, dX by itself, the pair, the sums / all
// three at once, the sums; a training pass' lower layer: 330 units, 21 rows of at most 97 frames, both directions, n_in = 660 19.5 + 18.6 + 13.0 / 31.8 + 5.1, n_in = 123 12.2 + 13.3 + 8.3 / 16.1 + 7.2;
// 208 units, 6 rows of 65 frames 11.1 + 11.2 + 5.0 / 12.0 + 5.0; 728 units, 14 rows of 113 frames, n_in = 598 19.3 + 26.2 + 13.0 / 37.7 + 4.3;
// 512 units, 32 rows of 60, both directions, n_in = 1024 23.6 + 34.6 + 6.8 / 48.8 + 4.0; 1000 units, 64 rows of 50, n_in = 1000 39.2 + 52.3 + 8.4 / 96.3 + 4.1).
hipError_t launch_gemm_tile_grads(const GemmArgs& dx, const GemmArgs& dwx, const GemmArgs& dwh, hipStream_t s) {
  const GemmArgs* g[3] = {&dx, &dwx, &dwh};
  for (int i = 0; i < 3; ++i)
    if (g[i]->M <= 0 || g[i]->N <= 0 || g[i]->nz <= 0) return hipErrorInvalidValue;
  const TileProduct p[3] = {sizes_of(dx), sizes_of(dwx), sizes_of(dwh)};
  int ks[3];
  tile_ranges3(p, dx.parts_bytes, ks);
  TileTrio a = {};
  size_t used = 0;
  for (int i = 0; i < 3; ++i) {
    a.p[i] = tile_args(*g[i], ks[i], used);
    used += tile_part_room(a.p[i].M, a.p[i].N, a.p[i].nz, a.p[i].ksplit);
  }
  const bool bf = dx.out_bf16 && a.p[0].ksplit == 1, rows = dwx.k_rows != nullptr;
  hipError_t e = bf ? (rows ? launch_grads_as<uint16_t, true>(a, s) : launch_grads_as<uint16_t, false>(a, s)) : rows ? launch_grads_as<float, true>(a, s) : launch_grads_as<float, false>(a, s);
  for (int i = 0; i < 3 && e == hipSuccess; ++i) e = finish(a.p[i], *g[i], s);
  return e;
}

}  // namespace lstm
