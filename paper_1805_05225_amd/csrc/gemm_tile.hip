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
// which also applies bias, row map and rounding.  (More stages in flight - three or four of them and one work-group per compute unit - were
// slower: 37 -> 49 us for 1600 x 4000 x 1000; a second work-group hides more than a deeper pipeline.)
//
// Operands go from global memory straight into LDS (16 bytes per lane), K in stages of 64, two stages; the order within a stage
// and the reasons are those of gemm_nt.hip.  A k-contiguous operand sits there as rows of 128 bytes whose 16-byte slot p holds
// chunk p ^ ((row / 2) % 8); a k-major one as 64 rows of one k each whose 64-byte blocks are XORed with k % 4, read with the LDS
// transpose read.
#include "recurrent_dev.h"
#include <algorithm>

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices
constexpr unsigned kParked = 0x7ffffff0u;
constexpr int kKB = 64;                 // k per stage

struct TileArgs {
  const char* A; const char* B; void* C; const float* bias;
  int M, N, K;
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

__device__ __forceinline__ void load_to_lds_b128(const u32x4& rsrc, unsigned lds_addr, unsigned voff, unsigned soff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ u32x4 make_rsrc(const void* base, long bytes) {
  const unsigned long long a = (unsigned long long)base;
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
  r[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane((unsigned)(bytes > 0x7fffff00L ? 0x7fffff00L : bytes));
  r[3] = kBufFlags;
  return r;
}
__device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Tile of WM x WN wavefronts, each TI x TJ blocks of 32 x 32.
template <int TI, int TJ, int WM, int WN>
struct Geo {
  static constexpr int kBM = WM * TI * 32, kBN = WN * TJ * 32, kNW = WM * WN;
  static constexpr int kOpA = kBM * kKB * 2, kOpB = kBN * kKB * 2, kStage = kOpA + kOpB;
  static constexpr int kLA = kOpA / 1024 / kNW, kLB = kOpB / 1024 / kNW;             // wavefront-loads per stage and wavefront
  static constexpr int kEpStride = kBN + 4, kEpBytes = WM * 32 * kEpStride * 4;      // the epilogue stages WM x 32 rows at a time
  static constexpr int kLds = 2 * kStage > kEpBytes ? 2 * kStage : kEpBytes;
};

// KROWS: k-major operands whose row k is row k_rows[k] in memory.
template <typename TC, bool AK, bool BK, bool KROWS, int TI, int TJ, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void gemm_tile_kernel(TileGroup grp) {
  typedef Geo<TI, TJ, WM, WN> G;
  constexpr int kBM = G::kBM, kBN = G::kBN, NW = G::kNW, kOpA = G::kOpA, kStage = G::kStage, kLA = G::kLA, kLB = G::kLB;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const bool second = (int)blockIdx.x >= grp.first1;
  const TileArgs g = second ? grp.p[1] : grp.p[0];
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int r = lane & 31, gq = lane >> 5;

  // bands of 8 tile columns, row-major inside a band: work-groups are dealt to the 8 XCDs round-robin, so each keeps one tile
  // column of B in its L2
  const int M = g.m_dev ? min(g.M, *g.m_dev) : g.M, K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  const int tiles_m = (g.M + kBM - 1) / kBM, tiles_n = (g.N + kBN - 1) / kBN;
  const int mine = (int)blockIdx.x - (second ? grp.first1 : 0), zk = mine / (tiles_m * tiles_n), bid = mine - zk * (tiles_m * tiles_n);
  const int band = bid / (8 * tiles_m), width = min(8, tiles_n - band * 8), rel = bid - band * 8 * tiles_m;
  const int m0 = __builtin_amdgcn_readfirstlane((rel / width) * kBM), n0 = __builtin_amdgcn_readfirstlane((band * 8 + rel % width) * kBN);
  if (m0 >= M) return;
  const int ksplit = g.ksplit, z = __builtin_amdgcn_readfirstlane(zk / ksplit), ks = __builtin_amdgcn_readfirstlane(zk - z * ksplit);

  const int ktiles = (K + kKB - 1) / kKB, nstage = ktiles * g.nseg;
  const int tail_chunks = (K - (ktiles - 1) * kKB + 7) >> 3;   // 16-byte chunks of a k-contiguous operand in the last k-tile
  // (told to be wave-uniform: divisions leave them in vector registers)
  const int it0 = __builtin_amdgcn_readfirstlane(nstage * ks / ksplit), total = __builtin_amdgcn_readfirstlane(nstage * (ks + 1) / ksplit) - it0;

  // k-contiguous operand, wavefront-load i: rows 8 (i NW + wave) .. + 7, lane l slot l & 7 of row l >> 3.
  // k-major operand, wavefront-load i: k-rows (i NW + wave) RPL .. + RPL - 1 of the stage, lane l slot l % (64 / RPL).
  constexpr int kRplA = 512 / kBM, kRplB = 512 / kBN;          // k-rows per load
  unsigned va[kLA], vb[kLB];
  bool pa[kLA], pb[kLB];                                       // k-contiguous: this lane's chunk lies past a ragged last k-tile
  const int ka_lane = lane / (64 / kRplA), kb_lane = lane / (64 / kRplB);
  const auto clip = [](long o, bool ok) { return ok && o <= 0x7ffffe00L ? (unsigned)o : kParked; };
#pragma unroll
  for (int i = 0; i < kLA; ++i) {
    pa[i] = false;
    if constexpr (AK) {
      const int rl = (i * NW + wave) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((rl >> 1) & 7);
      const int row = m0 + rl;
      const long pr = row < M ? (g.a_rows ? (long)g.a_rows[row] : row) : -1;
      va[i] = clip(pr * g.lda * 2 + chunk * 16, pr >= 0);
      pa[i] = chunk >= tail_chunks;
    } else {
      const int kk = (i * NW + wave) * kRplA + ka_lane, chunk = (lane % (64 / kRplA)) ^ (4 * (kk & 3));
      va[i] = clip((KROWS ? 0L : kk * g.lda * 2) + ((long)m0 + chunk * 8) * 2, m0 + chunk * 8 < M);
    }
  }
#pragma unroll
  for (int i = 0; i < kLB; ++i) {
    pb[i] = false;
    if constexpr (BK) {
      const int rl = (i * NW + wave) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((rl >> 1) & 7);
      const int row = n0 + rl;
      vb[i] = clip((long)row * g.ldb * 2 + chunk * 16, row < g.N);
      pb[i] = chunk >= tail_chunks;
    } else {
      const int kk = (i * NW + wave) * kRplB + kb_lane, chunk = (lane % (64 / kRplB)) ^ (4 * (kk & 3));
      vb[i] = clip((KROWS ? 0L : kk * g.ldb * 2) + ((long)n0 + chunk * 8) * 2, n0 + chunk * 8 < g.N);
    }
  }
  const int KB = AK && !BK && g.k_phys_rows > 0 ? g.k_phys_rows : K;
  const long k_mem = KROWS ? g.k_phys_rows : KB;
  const long a_bytes = (AK ? (long)(g.a_rows ? g.a_phys_rows : M) : k_mem) * g.lda * 2, b_bytes = (BK ? (long)g.N : k_mem) * g.ldb * 2;
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;

  // The stage whose loads go out next: segment, k-tile inside it (counted up, not divided out), and, with KROWS, the memory rows of
  // its k: entries of the packed list, by scalar loads that are waited for together with the operand loads (see gemm_nt.hip).  The
  // list is readable up to the next multiple of 64 entries.
  int seg = g.nseg > 1 ? __builtin_amdgcn_readfirstlane(it0 / ktiles) : 0, kt = it0 - seg * ktiles, left = total;
  u32x4 ra = make_rsrc(g.A + (g.sAz * z + g.sAseg * seg) * 2, a_bytes), rb = make_rsrc(g.B + (g.sBz * z + g.sBseg * seg) * 2, b_bytes);
  static_assert(!KROWS || (!AK && !BK && kLA == 4 && kRplA == 4 && kRplB == 4 && kLA == kLB), "four entries of the list per load, the same for A and B");
  i32x4 prow[KROWS ? kLA : 1];
  auto lookup = [&]() __attribute__((always_inline)) {         // for the stage that `kt` names
    if constexpr (KROWS) {
      if (left > 0) {
#pragma unroll
        for (int i = 0; i < kLA; ++i) {
          const int* p = g.k_rows + (long)kt * kKB + (i * NW + wave) * 4;
          asm volatile("s_load_dwordx4 %0, %1, 0x0" : "=s"(prow[i]) : "s"(p) : "memory");
        }
      }
    }
  };
  // Waits for the operand loads and the look-up.  The statement "rewrites" the entries, so that nothing that uses them is scheduled in
  // front of it (the compiler does not know that they are still on their way).
  auto wait_all = [&]() __attribute__((always_inline)) {
    if constexpr (KROWS) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+s"(prow[0]), "+s"(prow[1]), "+s"(prow[2]), "+s"(prow[3])::"memory");
    else __builtin_amdgcn_s_waitcnt(0x0070);                   // vmcnt(0) lgkmcnt(0)
  };
  const unsigned lda2 = (unsigned)g.lda * 2u, ldb2 = (unsigned)g.ldb * 2u;
  const unsigned odd = (ka_lane & 1) ? ~0u : 0u, high = (ka_lane & 2) ? ~0u : 0u;        // which of a load's four entries is this lane's
  auto issue = [&](int buf, int first, int last) __attribute__((always_inline)) {
    const bool tail = kt == ktiles - 1;
    const int k_left = KB - kt * kKB;                          // rows of a k-major operand from here on
    const unsigned dst = lds_base + buf * kStage + wave * 1024;
    const unsigned soA = AK ? (unsigned)kt * (kKB * 2) : KROWS ? 0u : (unsigned)kt * (kKB * lda2);
    const unsigned soB = BK ? (unsigned)kt * (kKB * 2) : KROWS ? 0u : (unsigned)kt * (kKB * ldb2);
#pragma unroll
    for (int q = 0; q < kLA + kLB; ++q) {
      if (q < first || q >= last) continue;
      const bool is_a = q < kLA;
      const int i = is_a ? q : q - kLA;
      unsigned v = is_a ? va[is_a ? i : 0] : vb[is_a ? 0 : i];
      if (is_a ? AK : BK) {
        if (tail && (is_a ? pa[is_a ? i : 0] : pb[is_a ? 0 : i])) v = kParked;
      } else {
        const bool ok = (i * NW + wave) * (is_a ? kRplA : kRplB) + (is_a ? ka_lane : kb_lane) < k_left;
        if constexpr (KROWS) {                                 // (32-bit arithmetic: the operands end below 2^31; a parked column stays past the end)
          const i32x4 p4 = prow[KROWS ? i : 0];
          const unsigned lo = ((unsigned)p4[0] & ~odd) | ((unsigned)p4[1] & odd), hi = ((unsigned)p4[2] & ~odd) | ((unsigned)p4[3] & odd);
          const unsigned row = (lo & ~high) | (hi & high);
          v = row * (is_a ? lda2 : ldb2) + v;
        }
        if (!ok) v = kParked;
      }
      load_to_lds_b128(is_a ? ra : rb, dst + (is_a ? 0 : kOpA) + i * NW * 1024, v, is_a ? soA : soB);
    }
  };
  auto advance = [&]() __attribute__((always_inline)) {        // every load of a stage has been issued
    --left;
    if (++kt == ktiles && AK && BK) {
      kt = 0;
      ++seg;
      ra = make_rsrc(g.A + (g.sAz * z + g.sAseg * seg) * 2, a_bytes);
      rb = make_rsrc(g.B + (g.sBz * z + g.sBseg * seg) * 2, b_bytes);
    }
  };

  // Fragments of k-step s (16 k): k-contiguous: row r of a block, chunk 2 s + gq; k-major: two transpose reads (see gemm_nt.hip).
  const int kc_off = r * 128 + ((gq ^ ((r >> 1) & 7)) * 16);
  const int l16 = lane & 15, sw = (l16 >> 2) & 3;
  const int km_row = gq * 8 + (l16 >> 2), km_low = ((lane >> 4) & 1) * 32 + (l16 & 3) * 8;
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  auto tr_read = [&](const char* p, int row_bytes) __attribute__((always_inline)) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * row_bytes));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    return make_uint4(l2.x, l2.y, h2.x, h2.y);
  };
  uint4 fa[2][TI], fb[2][TJ];
  auto read_frags = [&](int buf, int s, int c) __attribute__((always_inline)) {
    const char* base = lds + buf * kStage;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if constexpr (AK) fa[c][i] = *(const uint4*)(base + (wm * TI + i) * 32 * 128 + (kc_off ^ (s * 32)));
      else fa[c][i] = tr_read(base + (s * 16 + km_row) * (kBM * 2) + ((((wm * TI + i) ^ sw) & (kBM / 32 - 1)) << 6) + km_low, kBM * 2);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      if constexpr (BK) fb[c][j] = *(const uint4*)(base + kOpA + (wn * TJ + j) * 32 * 128 + (kc_off ^ (s * 32)));
      else fb[c][j] = tr_read(base + kOpA + (s * 16 + km_row) * (kBN * 2) + ((((wn * TJ + j) ^ sw) & (kBN / 32 - 1)) << 6) + km_low, kBN * 2);
    }
  };
  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  constexpr int NQ = kLA + kLB, kPer = (NQ + TI * TJ - 1) / (TI * TJ);      // loads behind each MFMA of the last k-step
  auto kstep = [&](int c, bool ld, int ld_buf) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < TI * TJ; ++m) {
      acc[m / TJ][m % TJ] = mma(fa[c][m / TJ], fb[c][m % TJ], acc[m / TJ][m % TJ]);
      if (ld) issue(ld_buf, m * kPer, (m + 1) * kPer < NQ ? (m + 1) * kPer : NQ);
    }
  };

  if (total > 0) {
    lookup();
    if constexpr (KROWS) wait_all();
    issue(0, 0, NQ);
    advance();
    lookup();
    wait_all();
    __syncthreads();
    if (total > 1) {
      issue(1, 0, NQ);
      advance();
      lookup();
    }
    read_frags(0, 0, 0);
  }
  for (int it = 0; it < total; ++it) {
    const int cur = it & 1;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      read_frags(cur, s + 1, (s + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      kstep(s & 1, false, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (it + 1 < total) {
      wait_all();                                              // own loads of stage it+1 (and row look-ups) landed, own reads of this stage done
      __syncthreads();
      read_frags(cur ^ 1, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (it + 2 < total) {
      kstep(1, true, cur);
      advance();
      lookup();
    } else {
      kstep(1, false, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // Epilogue: 32 rows of every wavefront row at a time through LDS, out as whole rows.
  constexpr int kEpStride = G::kEpStride, kTpr = kBN / 4;       // threads per row
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
  for (int i = 0; i < TI; ++i) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) ep[(wm * 32 + 8 * (v >> 2) + 4 * gq + (v & 3)) * kEpStride + (wn * TJ + j) * 32 + r] = acc[i][j][v];
    __syncthreads();
    if (col < g.N) {
      constexpr int kStep = 64 * NW / kTpr, kIts = WM * 32 / kStep;
      int crow[kIts];                                          // (looked up before the first store: a load behind a store waits for it)
#pragma unroll
      for (int q = 0; q < kIts; ++q) {
        const int rl = tid / kTpr + q * kStep, row = min(m0 + (rl >> 5) * TI * 32 + i * 32 + (rl & 31), M - 1);
        crow[q] = g.c_rows && !to_parts ? g.c_rows[row] : row;
      }
#pragma unroll
      for (int q = 0; q < kIts; ++q) {
        const int rl = tid / kTpr + q * kStep, row = m0 + (rl >> 5) * TI * 32 + i * 32 + (rl & 31);
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

template <typename TC, bool AK, bool BK, bool KROWS, int TI, int TJ, int WM, int WN>
hipError_t launch_as(const TileGroup& a, int count, hipStream_t s) {
  typedef Geo<TI, TJ, WM, WN> G;
  const auto kernel = gemm_tile_kernel<TC, AK, BK, KROWS, TI, TJ, WM, WN>;
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [&] { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, G::kLds); });
  if (ea != hipSuccess) return ea;
  TileGroup c = a;
  int blocks[2] = {0, 0};
  for (int i = 0; i < count; ++i) blocks[i] = cdiv(c.p[i].M, G::kBM) * cdiv(c.p[i].N, G::kBN) * c.p[i].nz * c.p[i].ksplit;
  c.first1 = count == 2 ? blocks[0] : 0x7fffffff;
  hipLaunchKernelGGL(kernel, dim3(blocks[0] + blocks[1]), dim3(64 * G::kNW), G::kLds, s, c);
  return hipGetLastError();
}
template <typename TC>
hipError_t launch_layout(const TileGroup& a, int count, bool ak, bool bk, hipStream_t s) {
  if (ak && bk) return launch_as<TC, true, true, false, 2, 2, 2, 2>(a, count, s);
  if (ak) return launch_as<TC, true, false, false, 2, 2, 2, 2>(a, count, s);
  if (a.p[0].k_rows) return launch_as<TC, false, false, true, 2, 2, 2, 2>(a, count, s);
  return launch_as<TC, false, false, false, 2, 2, 2, 2>(a, count, s);
}

long tiles_of(const GemmArgs& g) { return (long)cdiv(g.M, 128) * cdiv(g.N, 128) * g.nz; }
// `others`: tiles of the product that shares the launch
int ranges(long tiles, long others, long K, int nseg) {
  const long stages = (long)cdiv(K, kKB) * nseg;
  return (int)std::max(1L, std::min(std::min(512 / std::max(tiles + others, 1L), stages / 4), 16L));
}
size_t bytes_of(long M, long N, int nz, int ks) { return ks > 1 ? (size_t)ks * nz * M * ((N + 3) / 4 * 4) * 4 : 0; }
TileArgs tile_args(const GemmArgs& g, long others, size_t parts_used) {
  TileArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz;
  a.nseg = g.nseg; a.sAseg = g.sAseg; a.sBseg = g.sBseg; a.accumulate = g.accumulate;
  a.a_rows = g.a_rows; a.c_rows = g.c_rows; a.a_phys_rows = g.a_phys_rows; a.k_rows = g.k_rows; a.k_phys_rows = g.k_phys_rows;
  a.m_dev = g.m_dev; a.k_dev = g.k_dev;
  a.ldp = (g.N + 3) / 4 * 4;
  a.ksplit = g.parts ? ranges(tiles_of(g), others, g.K, g.nseg) : 1;
  if (parts_used + bytes_of(g.M, g.N, g.nz, a.ksplit) > g.parts_bytes) a.ksplit = 1;
  a.parts = a.ksplit > 1 ? (float*)((char*)g.parts + parts_used) : nullptr;
  return a;
}
hipError_t finish(const TileArgs& a, const GemmArgs& g, hipStream_t s) {
  if (a.ksplit == 1) return hipGetLastError();
  SumJob j = {};
  j.parts = a.parts; j.C = a.C; j.bias = a.bias; j.M = a.M; j.N = a.N; j.ksplit = a.ksplit; j.nz = a.nz;
  j.ldp = a.ldp; j.sPz = (long)a.ksplit * a.M * a.ldp; j.ldc = a.ldc; j.sCz = a.sCz; j.sbiasz = a.sbiasz;
  j.c_rows = a.c_rows; j.m_dev = a.m_dev; j.accumulate = a.accumulate; j.out_bf16 = g.out_bf16;
  return finish_parts(j, bytes_of(a.M, a.N, a.nz, a.ksplit), g.sums, s);
}

}  // namespace

bool gemm_tile_ok(const GemmArgs& g) {
  const auto a16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  const long lim = 0x7ffffe00L;           // operands are addressed with 32-bit byte offsets
  const long k_rows = g.k_phys_rows > 0 ? g.k_phys_rows : g.K, a_rows = g.a_kcontig ? (g.a_rows ? g.a_phys_rows : g.M) : k_rows;
  if (a_rows * g.lda * 2 > lim || (g.b_kcontig ? (long)g.N : k_rows) * g.ldb * 2 > lim) return false;
  if (g.a_kcontig && (g.K % 8 != 0 || (g.k_dev && g.K % 64 != 0))) return false;   // whole chunks; a device-resident K counts whole stages there
  if (!g.a_kcontig && (g.b_kcontig || g.a_rows || g.m_dev || g.nseg > 1)) return false;
  if (g.a_kcontig && !g.b_kcontig && (g.k_rows || g.nseg > 1)) return false;
  return g.in_bf16 && !g.lens && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.sAz % 8 == 0 && g.sBz % 8 == 0 && g.sAseg % 8 == 0 && g.sBseg % 8 == 0 &&
         a16(g.A) && a16(g.B) && !(g.accumulate && g.out_bf16);
}

// Fewer 256 x 256 tiles than fill the device's 256 compute units: those of gemm_nt.hip would leave some idle for the whole product.  The line
// lies between 192 tiles (1600 real of 3000 rows x 4000 x 1000: 55 us there, 24 here) and 237 (768 x 20000 x 1000: 44 us there, 49 here).
bool gemm_tile_small(long M, long N, int nz) { return (long)cdiv(M, 256) * cdiv(N, 256) * nz <= 200; }

size_t gemm_tile_parts_bytes(long M, long N, long K, int nz, int nseg) {
  return bytes_of(M, N, nz, ranges((long)cdiv(M, 128) * cdiv(N, 128) * nz, 0, K, nseg));
}

hipError_t launch_gemm_tile(const GemmArgs& g, hipStream_t s) {
  TileGroup a = {};
  a.p[0] = tile_args(g, 0, 0);
  const bool bf = g.out_bf16 && a.p[0].ksplit == 1;
  const hipError_t e = bf ? launch_layout<uint16_t>(a, 1, g.a_kcontig, g.b_kcontig, s) : launch_layout<float>(a, 1, g.a_kcontig, g.b_kcontig, s);
  return e == hipSuccess ? finish(a.p[0], g, s) : e;
}

// dW_x and dW_h: each alone leaves the device's last work-groups waiting for it, and wants twice the K ranges to fill the device.
hipError_t launch_gemm_tile_pair(const GemmArgs& g, const GemmArgs& h, hipStream_t s) {
  if (g.M <= 0 || h.M <= 0 || g.N <= 0 || h.N <= 0 || g.nz <= 0) return hipErrorInvalidValue;
  TileGroup a = {};
  a.p[0] = tile_args(g, tiles_of(h), 0);
  a.p[1] = tile_args(h, tiles_of(g), (bytes_of(g.M, g.N, g.nz, a.p[0].ksplit) + 255) / 256 * 256);
  hipError_t e = launch_layout<float>(a, 2, false, false, s);
  if (e != hipSuccess || (e = finish(a.p[0], g, s)) != hipSuccess) return e;
  return finish(a.p[1], h, s);
}

}  // namespace lstm
