// Products with few rows (M <= about a thousand): the stepped decoder cell (Sec. 7, Listing 1: "s", an LSTM cell fed by
// 620 + 2000 values for 64 sentences x beam 12 = 768 rows), and the linear layers around it ("s_tr", "readout", the
// output layer).  The throughput kernels of gemm_nt.hip use 256 x 256 tiles: 768 rows x 4000 columns are 48 tiles, so
// K had to be cut into ranges whose partial products went through memory (61 MB per step) and a second pass.  Here a
// work-group owns 96 rows x 128 columns - 768 x 4096 is exactly 256 tiles, one per compute unit - and walks the
// whole K, so the result is complete in the work-group and the epilogue can finish the job:
//   * plain:  C = A B^T + bias, optionally max(0, .), float or bfloat16;
//   * cell:   the 128 columns are the four gates of 32 hidden units (the packed weights are ordered that way), and
//             the epilogue adds the bias, applies the LSTM cell and writes y, h', c' - no pre-activations in memory.
//
// C[M,N] = A[M,K] B[N,K]^T, both operands bfloat16, k-contiguous, rows 16-byte aligned, K a multiple of 8.
// Eight wavefronts: wavefront (kq, wc) owns the 96 x 64 block of column half wc (3 x 2 MFMA blocks of 32x32x16) for
// k-step kq of every 64-wide stage (five fragment reads for six MFMAs; with 96 x 32 per wavefront the LDS reads took
// longer than the MFMAs); the four shares are added in the epilogue.  Two wavefronts per SIMD.  Operands travel from global memory straight into LDS (16 bytes
// per lane, 1 KiB per wavefront instruction = 8 rows of 128 bytes), four stages of 64 k, one barrier per stage; bank conflicts
// are avoided by placement: the 16-byte slot p of row r holds k-chunk p ^ ((r >> 1) & 7).  What bounds it is the path
// from L2 to LDS (about 47 bytes per clock and compute unit, measured for the large kernels): 28 KiB per stage
// against 384 clocks of MFMA work, i.e. about 600 clocks per stage.
//
// Other tile shapes (64 x 64: every wavefront one k-step of a 64 x 32 block) serve products that 96 x 128 tiles would leave compute units
// without (the decoder's query projection and readout, 768 x 1000: 64 tiles against 192) or take a second round for: what bounds the kernel is the
// rate at which ONE compute unit pulls operands from L2, so more, smaller tiles finish sooner although they move more bytes in total (launch_tiles).
#include "recurrent_dev.h"
#include "gemm_skinny.h"

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices
constexpr int kRow = 128;                          // bytes per LDS row (64 bfloat16)
constexpr int kDepth = 4;                          // stages in LDS: three in flight while one is multiplied (2: +20 %, 3 and 5: the same)
// Tile geometry for wavefront blocks of BI x BJ MFMA blocks (32 x 32): the tile is 32 BI rows x 64 BJ columns.
template <int BI, int BJ>
struct Geo {
  static constexpr int kTM = 32 * BI, kTN = 64 * BJ;
  static constexpr int kAop = kTM * kRow, kBop = kTN * kRow, kStage = kAop + kBop;   // <3,2>: 12 + 16 KiB
  static constexpr int kLoads = (kTM + kTN) / 8;                                      // wavefront-loads per stage
  static constexpr int kPerWave = (kLoads + 7) / 8;                                   // issued by every wavefront per stage
  static constexpr int kDummy = kDepth * kStage;      // 4 KiB that the surplus loads of a stage write zeros to (see the kernel)
  static constexpr int kEpStride = kTN + 4;           // floats per staged row
  static constexpr int kLds = kDummy + 4096;          // <3,2>: 118784 bytes; the epilogue's staging reuses the stages
  static_assert(2 * kTM * kEpStride * 4 <= kLds, "the epilogue's staging (no load is in flight then)");
};
constexpr unsigned kParked = 0x7ffffff0u;

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
__device__ __forceinline__ f32x16 mma32(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// s_waitcnt operand for vmcnt(n) lgkmcnt(0): vmcnt's low four bits sit in bits 3:0, its upper two in bits 15:14
constexpr int vm_wait(unsigned n) { return (int)(0x0070u | (n & 15u) | ((n >> 4) << 14)); }

// Work-group -> tile.  Work-groups are dealt to the eight XCDs round-robin (blockIdx & 7 is the XCD).  An XCD's tiles are a rectangle of
// pr x pc of them, xr rectangles over the rows, 8 / xr over the columns: what its L2 has to fetch are pr row and pc column panels, so
// xr is where these are fewest bytes, after the number of rounds (of 32 work-groups an XCD) that the largest rectangle takes.
// What comes from beyond L2 arrives at a quarter of the rate of what is in it (11 against 47 bytes a clock and compute unit), and the two
// add up: 768 x 1000 x 3620 in 64 x 64 tiles, 12 x 2 of them an XCD (every row of A in every L2, 7.2 MB) 21.5 us, 6 x 4 (5 MB) 20.2.
struct Tile { int tm, tn, pos; bool live; };
__device__ __forceinline__ Tile tile_of(const SkinnyArgs& g, int tiles_m, int tiles_n) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, across = slot / g.pr, down = slot - across * g.pr;
  Tile t;
  t.tm = (xcd & (g.xr - 1)) * g.pr + down; t.tn = xcd / g.xr * g.pc + across; t.pos = slot & 31;
  t.live = t.tm < tiles_m && t.tn < tiles_n;
  return t;
}
// xr, pr, pc for tiles of tm x tn; the rounds, of all nz problems
int split_tiles(SkinnyArgs& a, int tm, int tn) {
  const int tiles_m = cdiv(a.M, tm), tiles_n = cdiv(a.N, tn);
  long best = 0;
  int rounds = 0;
  for (int xr = 1; xr <= 8; xr *= 2) {
    const int pr = cdiv(tiles_m, xr), pc = cdiv(tiles_n, 8 / xr), r = cdiv((long)pr * pc * a.nz, 32);
    const long cost = ((long)r << 32) + (long)pr * tm + (long)pc * tn;
    if (xr == 1 || cost < best) { best = cost; rounds = r; a.xr = xr; a.pr = pr; a.pc = pc; }
  }
  return rounds;
}

// BFRAG: B in fragment order, [row tile of 16][g.b_nkc chunks of 32 k][64 lanes] of 16 bytes (launch_pack_rows_both), a wavefront-load is a chunk of a tile.
template <int BI, int BJ, bool CELL, bool BFRAG>
__global__ __launch_bounds__(512) void skinny_kernel(SkinnyArgs g) {
  typedef Geo<BI, BJ> G;
  constexpr int kTM = G::kTM, kTN = G::kTN, kAop = G::kAop, kStage = G::kStage, kLoads = G::kLoads, kDummy = G::kDummy,
                kEpStride = G::kEpStride, kPerWave = G::kPerWave;
  constexpr int kUnits = 16 * BJ;                   // cell: the tile's columns are the four gates of so many units
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = wave >> 1, wc = wave & 1;          // k-step of a stage (0..3) and column half (32 BJ columns) of this wavefront
  const int r = lane & 31, gq = lane >> 5;
  const int tiles_m = (g.M + kTM - 1) / kTM, tiles_n = (g.N + kTN - 1) / kTN;
  const Tile tl = tile_of(g, tiles_m, tiles_n);
  if (!tl.live) return;
  const int m0 = tl.tm * kTM, n0 = tl.tn * kTN, z = blockIdx.z;
  const int K = g.K, nstage = (K + 63) / 64;
  // The work-groups of an XCD that share an operand panel would ask for the same lines at the same time, and all of them would wait for the one
  // fetch from beyond L2.  So they start a little apart, an eighth of K between the first and the last of the 32 that an XCD runs together, and wrap around
  // (a sum's order follows from its work-group's position alone: the same call gives the same bits).  Not further: operands of 9 MB per XCD do not stay in 4 MB of L2 until the last
  // of them comes by (over all of K, half of the decoder cell's requests missed: 768 rows, K = 3620, N = 4000 39.9 us, 37.8 so; 37.3 with no
  // distance at all, but up to 2 % more for 640 rows and less).
  const int rot = (int)(((long)tl.pos * nstage) >> 8);

  f32x16 acc[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Loads: wavefront-load q of a stage (q = wave + 8 i) fills rows 8 q' .. 8 q' + 7 of A (q < kTM / 8) or B (q < kLoads);
  // lane l fills slot l & 7 of row l >> 3 of those, i.e. fetches k-chunk (l & 7) ^ swizzle(row).  Rows past the operand's
  // end and chunks past K point outside the buffer descriptor and arrive as zeros.  Every wavefront issues the same
  // number of loads per stage, so that one wait count serves all of them: surplus ones (q >= kLoads; four in the 96 x 128
  // tile) have every lane parked and write their zeros to a spare 4 KiB of LDS without touching memory.
  unsigned voff[kPerWave], dst[kPerWave];
  int chunk[kPerWave];
  bool is_b[kPerWave];
  const long a_bytes = (long)g.M * g.lda * 2, b_bytes = BFRAG ? (long)((g.N + 15) / 16) * g.b_nkc * 1024 : (long)g.N * g.ldb * 2;
#pragma unroll
  for (int i = 0; i < kPerWave; ++i) {
    const int q = wave + 8 * i;
    const bool real = q < kLoads;
    is_b[i] = q >= kTM / 8;
    const int rg = is_b[i] ? q - kTM / 8 : q;
    const int rl = rg * 8 + (lane >> 3);
    chunk[i] = real ? (lane & 7) ^ ((rl >> 1) & 7) : 0x10000;            // surplus load: "past K" in every stage
    // (packed rows of the cell come in blocks of 32 units: 128 t + 32 gate + unit)
    const int b_row = CELL ? 128 * (tl.tn * kUnits >> 5) + 32 * (rl / kUnits) + (tl.tn * kUnits & 31) + rl % kUnits : n0 + rl;
    const long row = is_b[i] ? b_row : m0 + rl;
    bool inside = real && (is_b[i] ? row < g.N : row < g.M);
    long off = row * (is_b[i] ? g.ldb : g.lda) * 2 + (chunk[i] & 7) * 16;
    if (BFRAG && real && is_b[i]) {                                      // (rows that fill up the last tile are zeros)
      const int tile = (n0 >> 4) + (rg >> 1);
      inside = tile * 16 < g.N;
      chunk[i] = 4 * (rg & 1);
      off = ((long)tile * g.b_nkc + (rg & 1)) * 1024 + lane * 16;
    }
    voff[i] = (inside && off <= 0x7fffff00L) ? (unsigned)off : kParked;
    dst[i] = real ? (unsigned)((is_b[i] ? kAop : 0) + rg * 1024) : 0u;
  }
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)lds;
  const u32x4 ra = make_rsrc(g.A + g.sAz * z * 2, a_bytes > 0x7fffff00L ? 0x7fffff00u : (unsigned)a_bytes);
  const u32x4 rb = make_rsrc(g.B + g.sBz * z * 2, b_bytes > 0x7fffff00L ? 0x7fffff00u : (unsigned)b_bytes);
  auto issue = [&](int it) __attribute__((always_inline)) {
    const unsigned buf = lds_base + (unsigned)(it % kDepth) * kStage;
    const int kt = it + rot < nstage ? it + rot : it + rot - nstage;       // which 64 k this stage holds
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) {
      const bool past = kt * 64 + chunk[i] * 8 >= K;           // ragged last k-tile (and every surplus load; K: up to whole chunks of 32 with BFRAG)
      const unsigned where = wave + 8 * i >= kLoads ? lds_base + kDummy + (unsigned)(wave & 3) * 1024u : buf + dst[i];
      load_to_lds_b128(is_b[i] ? rb : ra, where, past ? kParked : voff[i], (unsigned)kt * (BFRAG && is_b[i] ? 2048u : 128u));
    }
  };
  // Fragment reads: row (i*32 + r) of A / (wc*32*BJ + j*32 + r) of B, k-chunk 2 kq + gq, in slot (2 kq + gq) ^ ((row >> 1) & 7)
  const int slot = ((2 * kq + gq) ^ ((r >> 1) & 7)) * 16;
  const int fa_off = r * kRow + slot;
  // (BFRAG: 2 KiB per tile of 16 columns; lanes of a chunk lie side by side)
  const int fb_off = kAop + (BFRAG ? wc * 2 * BJ * 2048 + (r >> 4) * 2048 + ((2 * kq + gq) * 16 + (r & 15)) * 16 : (wc * 32 * BJ + r) * kRow + slot);

  // Pipeline: while the MFMAs of stage it run (fragments in registers), the fragments of stage it+1 are read from LDS
  // and the loads of stages it+2 .. it+4 are in flight (a load from beyond L2 takes longer than two stages of MFMAs:
  // with one stage ahead the loop ran at memory latency, 1700 clocks per stage; and with fragment reads and MFMAs of
  // one stage in program order the compiler made every MFMA wait for its own LDS read).  Loads complete in issue
  // order, four per wavefront and stage: when at most 8 are outstanding, everything up to the stage two behind the
  // newest has landed.  A buffer is overwritten one iteration after every wavefront has passed the barrier behind
  // which it read the buffer's fragments (and waited for them).
  uint4 fa[2][BI], fb[2][BJ];                      // [register set][row block], [register set][column block]
  auto read_a = [&](int it, int set, int i) __attribute__((always_inline)) {
    fa[set][i] = *(const uint4*)(lds + (it % kDepth) * kStage + fa_off + i * 32 * kRow);
  };
  auto read_b = [&](int it, int set, int j) __attribute__((always_inline)) {
    fb[set][j] = *(const uint4*)(lds + (it % kDepth) * kStage + fb_off + j * 32 * kRow);
  };
  auto wait_stage = [&](int newer) __attribute__((always_inline)) {       // `newer` stages were issued behind the awaited one
    if (newer >= 4) __builtin_amdgcn_s_waitcnt(vm_wait(4 * kPerWave));
    else if (newer == 3) __builtin_amdgcn_s_waitcnt(vm_wait(3 * kPerWave));
    else if (newer == 2) __builtin_amdgcn_s_waitcnt(vm_wait(2 * kPerWave));
    else if (newer == 1) __builtin_amdgcn_s_waitcnt(vm_wait(kPerWave));
    else __builtin_amdgcn_s_waitcnt(vm_wait(0));
  };
#pragma unroll
  for (int j = 0; j < kDepth; ++j)
    if (j < nstage) issue(j);
  wait_stage(min(nstage - 1, kDepth - 1));
  __syncthreads();
  // fragment read number q of a stage, in the order the MFMAs will want them: B block 0, the A blocks, the other B blocks
  auto read_nr = [&](int it, int set, int q) __attribute__((always_inline)) {
    if (q == 0) read_b(it, set, 0);
    else if (q <= BI) read_a(it, set, q - 1);
    else if (q < BI + BJ) read_b(it, set, q - BI);
  };
  // The MFMAs of a stage in the order (row block, column block) = (0,0) (1,0) .. (0,1) (1,1) ..; with `next`, one
  // fragment read of the following stage goes out behind each MFMA (96 x 128 tile: behind the first five of six),
  // what is left of them behind the last.  (All reads in front of the MFMAs held the MFMAs back until the LDS had
  // taken them: reads and MFMAs of a stage then ran one after the other.)
  auto mfmas = [&](int set, bool next, int it_next) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < BI * BJ; ++m) {
      const int i = m % BI, j = m / BI;
      acc[i][j] = mma32(fa[set][i], fb[set][j], acc[i][j]);
      if (next) {
        __builtin_amdgcn_sched_barrier(0);
        read_nr(it_next, set ^ 1, m);
        if (m == BI * BJ - 1) {
#pragma unroll
          for (int q = BI * BJ; q < BI + BJ; ++q) read_nr(it_next, set ^ 1, q);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // one stage with a successor.  No branch between the successor's reads and the MFMAs: where two paths with different
  // numbers of pending LDS reads met in front of the MFMAs, the compiler made them wait for every read.
  auto step = [&](int it, int set) __attribute__((always_inline)) {
    wait_stage(min(nstage - 2 - it, kDepth - 2));                         // stage it+1 landed; own fragment reads of stage it done
    __syncthreads();
    if (it + kDepth < nstage) issue(it + kDepth);                         // into the buffer of stage it, now in registers everywhere
    __builtin_amdgcn_sched_barrier(0);
    mfmas(set, true, it + 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // (the last stage is in register set 1 whatever their number: two ends for two parities cost a second set of accumulators)
  int it = 0;
  if (nstage & 1) {
#pragma unroll
    for (int q = 0; q < BI + BJ; ++q) read_nr(0, 1, q);
    if (nstage > 1) step(it++, 1);
  } else {
#pragma unroll
    for (int q = 0; q < BI + BJ; ++q) read_nr(0, 0, q);
  }
  if (nstage > 1) {
    for (; it + 2 < nstage; it += 2) {
      step(it, 0);
      step(it + 1, 1);
    }
    step(it, 0);
  }
  if (nstage > 0) mfmas(1, false, 0);
  __syncthreads();                                 // the stage buffers are free for the epilogue

  // Epilogue.  The four k-steps' shares meet in LDS (the stage buffers are free): k-steps 2 and 3 store theirs side by side, 0 and 1
  // add to them, and whoever reads adds the two.  (One after the other into one array, four rounds of it, took 8 us of the 768-row
  // cell's 39.)  acc[i][j][v] is row i*32 + 8 (v / 4) + 4 gq + v % 4, column wc*32*BJ + j*32 + r.
  float* ep = (float*)lds;
  constexpr int kEpHalf = kTM * kEpStride;
#pragma unroll
  for (int round = 1; round >= 0; --round) {
    if ((kq >> 1) == round) {
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j, __builtin_amdgcn_sched_barrier(0))      // (one block's reads at a time)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float* e = &ep[(kq & 1) * kEpHalf + (i * 32 + 8 * (v >> 2) + 4 * gq + (v & 3)) * kEpStride + wc * 32 * BJ + j * 32 + r];
            *e = round == 1 ? acc[i][j][v] : *e + acc[i][j][v];
          }
    }
    __syncthreads();
  }
  if constexpr (!CELL) {
    // thread -> (row, four columns): kTN / 4 threads per row, 512 / (kTN / 4) rows per pass
    constexpr int kTpr = kTN / 4;
    const int c4 = (tid % kTpr) * 4, col = n0 + c4;
    const float* bias = g.bias ? g.bias + g.sbiasz * z : nullptr;
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
      for (int k = 0; k < 4; ++k) if (col + k < g.N) bv[k] = bias[col + k];
    }
    const bool vec = (g.ldc % 4 == 0) && ((((uintptr_t)g.C) & 15u) == 0) && (g.sCz % 4 == 0) && col + 3 < g.N;
    for (int rr = tid / kTpr; rr < kTM; rr += 512 / kTpr) {
      const int row = m0 + rr;
      if (row >= g.M || col >= g.N) continue;
      const float4 val = *(const float4*)&ep[rr * kEpStride + c4], val2 = *(const float4*)&ep[kEpHalf + rr * kEpStride + c4];
      float e[4] = {val.x + val2.x + bv[0], val.y + val2.y + bv[1], val.z + val2.z + bv[2], val.w + val2.w + bv[3]};
      if (g.relu) {
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = e[k] > 0.f ? e[k] : 0.f;
      }
      const long off = g.sCz * z + (long)row * g.ldc + col;
      if (g.out_bf16) {
        uint16_t* Cb = (uint16_t*)g.C + off;
        if (vec) {
          uint2 o;
          o.x = f2bf_bits(e[0]) | ((unsigned)f2bf_bits(e[1]) << 16);
          o.y = f2bf_bits(e[2]) | ((unsigned)f2bf_bits(e[3]) << 16);
          *(uint2*)Cb = o;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) if (col + k < g.N) Cb[k] = f2bf_bits(e[k]);
        }
      } else {
        float* Cf = (float*)g.C + off;
        if (vec) *(float4*)Cf = make_float4(e[0], e[1], e[2], e[3]);
        else {
#pragma unroll
          for (int k = 0; k < 4; ++k) if (col + k < g.N) Cf[k] = e[k];
        }
      }
    }
  } else {
    // thread -> (unit of the tile, row): a thread per unit and row, 512 / kUnits rows per pass; staged columns kUnits q + unit
    const int uu = tid % kUnits, j = tl.tn * kUnits + uu, n = g.n;
    if (tid == 0 && (blockIdx.x | blockIdx.z) == 0) *g.status = 0u;
    if (j < n) {
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (g.bias) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[q] = g.bias[(long)z * 4 * n + q * n + j];
      }
      for (int rr = tid / kUnits; rr < kTM; rr += 512 / kUnits) {
        const int b = m0 + rr;
        if (b >= g.M) break;
        const long si = ((long)z * g.M + b) * n + j;
        const bool valid = clamp_len(g.lens, b, 1) > 0;
        float c = g.c_in ? g.c_in[si] : 0.f, h = 0.f;
        if (valid) {
          float zh[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) zh[q] = ep[rr * kEpStride + q * kUnits + uu] + ep[kEpHalf + rr * kEpStride + q * kUnits + uu] + bv[q];
          const float zx[4] = {0.f, 0.f, 0.f, 0.f};
          const CellOut o = lstm_cell(zh, zx, c);
          c = o.c; h = o.h;
        }
        g.y[(long)b * g.ldy + (long)z * n + j] = f2bf_bits(h);
        if (g.cs) g.cs[si] = c;
        if (g.c_out) g.c_out[si] = c;
        if (g.h_out) g.h_out[si] = valid ? h : (g.h_in ? g.h_in[si] : 0.f);
      }
    }
  }
}

template <int BI, int BJ, bool CELL, bool BFRAG>
hipError_t launch_as(const SkinnyArgs& a, hipStream_t s) {
  typedef Geo<BI, BJ> G;
  static std::atomic<unsigned long long> attr_set{0};
  const hipError_t ea = once_per_device(attr_set, [] {
    return hipFuncSetAttribute((const void*)skinny_kernel<BI, BJ, CELL, BFRAG>, hipFuncAttributeMaxDynamicSharedMemorySize, G::kLds);
  });
  if (ea != hipSuccess) return ea;
  const dim3 grid(8 * a.pr * a.pc, 1, a.nz);
  hipLaunchKernelGGL((skinny_kernel<BI, BJ, CELL, BFRAG>), grid, dim3(512), G::kLds, s, a);
  return hipGetLastError();
}
constexpr int kTiles[][2] = {{3, 2}, {2, 1}, {2, 2}, {3, 1}, {4, 2}, {1, 1}};
int choose_tile(SkinnyArgs& a, double& least) {
  int best = 0;
  for (int i = 0; i < 6; ++i) {
    const int tm = 32 * kTiles[i][0], tn = 64 * kTiles[i][1];
    SkinnyArgs b = a;
    const double cost = split_tiles(b, tm, tn) * ((a.M < tm ? a.M : tm) + tn + 1e5 / a.K);
    if (i == 0 || cost < least) { least = cost; best = i; }
  }
  return best;
}
template <bool CELL, bool BFRAG>
hipError_t launch_tiles(SkinnyArgs a, hipStream_t s) {
  // The tile whose work-groups are done first: rounds times what one reads, which is all of K of its rows and columns; what begins and ends
  // a work-group counts as 1e5 / K rows more.  Of 46 products and cells measured with every tile the choice is the fastest one or within 6 %, in three
  // within 12 % (64 x 32000 x 512 12.2 us, 10.9 in 64 x 64).  us, 96 x 128 (or 64 x 64) before and the choice: cells of n = 688, 915 rows, K = 1680 44.9 -> 26.0; n = 1000, 1024 rows,
  // K = 3620 71.9 -> 49.0; n = 504, 504 rows, K = 2424 31.2 -> 19.8; both directions of a cell are one launch and share its rounds (over 237 such cells of more than 192 rows the choice is
  // 1.02 times the fastest tile in the mean, 1.09 with the rounds of one direction: 930 rows, n = 276, K = 2240 43.6 -> 34.6, 898 rows, n = 384, K = 2880 51.9 -> 42.0); products 1000 x 4000 x 2000 43.8 -> 30.2, 104 x 22051 x 960 29.8 -> 19.5, 504 x 920 x 2424 14.3 -> 12.5.
  double least = 0.;
  const int best = choose_tile(a, least);
  split_tiles(a, 32 * kTiles[best][0], 64 * kTiles[best][1]);
  switch (best) {
    case 0: return launch_as<3, 2, CELL, BFRAG>(a, s);
    case 1: return launch_as<2, 1, CELL, BFRAG>(a, s);
    case 2: return launch_as<2, 2, CELL, BFRAG>(a, s);
    case 3: return launch_as<3, 1, CELL, BFRAG>(a, s);
    case 4: return launch_as<4, 2, CELL, BFRAG>(a, s);
    default: return launch_as<1, 1, CELL, BFRAG>(a, s);
  }
}
hipError_t launch(const SkinnyArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.nz <= 0) return hipSuccess;
  if (a.cell) return launch_tiles<true, false>(a, s);
  if (a.b_nkc) return launch_tiles<false, true>(a, s);
  if (few_rows_pay(a.M, a.N, a.K)) return launch_few(a, s);
  return launch_tiles<false, false>(a, s);
}

// Wcell[d][128 t + 32 q + u][k] = [W_x^T | 0 | W_h^T | 0] row (q n + 32 t + u), zero for units past n; a 64 x 64 tile of
// (k, packed row) per work-group: rows of W are read along the packed-row axis in runs of 32 consecutive columns.
__global__ __launch_bounds__(256) void pack_wcell_kernel(const uint16_t* Wx, const uint16_t* Wh, uint16_t* Wc, int n_in, int n_in_pad, int n,
                                                         int Kc, int Np) {
  __shared__ uint16_t tile[64][66];
  const int N4 = 4 * n;
  const int d = blockIdx.z;
  Wx += (long)d * n_in * N4;
  Wh += (long)d * n * N4;
  Wc += (long)d * Np * Kc;
  const int k0 = blockIdx.x * 64, p0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  {
    const int p = p0 + tx, t = p >> 7, q = (p >> 5) & 3, u = p & 31, j = t * 32 + u;
    const int col = q * n + j;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int k = k0 + ty + 4 * i;
      uint16_t v = 0;
      if (p < Np && j < n) {
        if (k < n_in) v = Wx[(long)k * N4 + col];
        else if (k >= n_in_pad && k < n_in_pad + n) v = Wh[(long)(k - n_in_pad) * N4 + col];
      }
      tile[ty + 4 * i][tx] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int p = p0 + ty + 4 * i, k = k0 + tx;
    if (p < Np && k < Kc) Wc[(long)p * Kc + k] = tile[tx][ty + 4 * i];
  }
}

}  // namespace

// only where the 256 x 256 tiles of the throughput kernel would leave most of the device idle (it is the faster one
// from about half a device's worth of tiles: 768 x 20000 x 1000 takes 49 us there and 72 us here)
bool gemm_skinny_pays(long M, long N, int nz) { return M <= kSkinnyMaxRows && (long)cdiv(M, 256) * cdiv(N, 256) * nz < 128; }
bool gemm_skinny_ok(const GemmArgs& g) {
  const auto a16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  return gemm_skinny_pays(g.M, g.N, g.nz) && g.in_bf16 && g.a_kcontig && g.b_kcontig && !g.lens && g.nseg == 1 && !g.a_rows && !g.c_rows && !g.m_dev &&
         !g.k_dev && !g.accumulate && g.K % 8 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.sAz % 8 == 0 && g.sBz % 8 == 0 &&
         a16(g.A) && a16(g.B) && (long)g.N * g.ldb * 2 <= 0x7fffff00L;
}
// A work-group here begins and ends alone on its compute unit, one of 128 x 128 (gemm_tile.hip) shares it, and one of 256 x 256 (gemm_nt.hip) moves fewest bytes: with many columns the
// best of the three changes several times.  Each side as measured, in us, operands from memory, 20 to 1024 rows, 300 to 32000 columns, K from 272 to 8000 (691 products): the choice
// is the fastest or within 5 % in all but 20 of them, at most 1.33 times it; by the number of 256 x 256 tiles alone (here below 128, 128 x 128 up to 200) 134 were not, the
// worst 1.44.  us, here / 128 x 128 / 256 x 256: 224 x 20000 x 448 17.7 / 14.9 / 19.0, 385 x 14000 x 448 20.2 / 14.0 / 19.0, 480 x 20000 x 800 48.4 / 37.2 / 28.8, 600 x 9000 x 448 17.8 / 14.6 /
// 19.4, 300 x 5000 x 800 10.3 / 13.8 / 25.2, 900 x 5000 x 800 22.3 / 19.2 / 25.4.
FewRoute few_rows_route(int M, int N, int K) {
  SkinnyArgs a = {};
  a.M = M; a.N = N; a.K = K; a.nz = 1;
  double cost = 0.;
  const int best = choose_tile(a, cost), rounds = split_tiles(a, 32 * kTiles[best][0], 64 * kTiles[best][1]);
  const double out = 1e-6 * M * N, k = 1e-3 * K, read = rounds ? cost / rounds - 1e5 / K : 0.;      // rows and columns that a work-group reads
  const int groups = cdiv(M, 128) * cdiv(N, 128), full = (groups - 1) / 512, rest = groups - 512 * full, pairs = full + (rest > 256), alone = rest <= 256;
  const int large = cdiv((long)cdiv(M, 256) * cdiv(N, 256), 256);
  const double here = 2.0 + rounds * (1.63 + 0.034 * k * read) + 1.56 * out;
  const double tile = 2.8 + pairs * (1.63 + 16.6 * k) + alone * (4.1 + 7.1 * k) + 0.89 * out;
  const double nt = large * (10.2 + 16.4 * k) + 0.55 * out;
  return here <= tile && here <= nt ? FewRoute::kHere : tile <= nt ? FewRoute::kTile : FewRoute::kLarge;
}
hipError_t launch_gemm_skinny(const GemmArgs& g, hipStream_t s) {
  SkinnyArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz;
  a.out_bf16 = g.out_bf16;
  return launch(a, s);
}
hipError_t launch_skinny_readout(const void* A, long lda, const void* Wfrag, const float* bias, void* out, long ldo, int B, int R, int K, hipStream_t s) {
  SkinnyArgs a = {};
  a.A = (const char*)A; a.B = (const char*)Wfrag; a.C = out; a.bias = bias;
  a.b_nkc = cdiv(K, 32);
  a.M = B; a.N = R; a.K = 32 * a.b_nkc; a.lda = lda; a.ldc = ldo; a.nz = 1;
  a.out_bf16 = 1; a.relu = 1;
  return launch(a, s);
}
hipError_t launch_pack_wcell(const void* W_x, const void* W_h, void* Wcell, int n_in, int n_in_pad, int n, int Kc, int ndir, hipStream_t s) {
  const int Np = 128 * cdiv(n, 32);
  hipLaunchKernelGGL(pack_wcell_kernel, dim3(cdiv(Kc, 64), cdiv(Np, 64), ndir), dim3(256), 0, s, (const uint16_t*)W_x, (const uint16_t*)W_h,
                     (uint16_t*)Wcell, n_in, n_in_pad, n, Kc, Np);
  return hipGetLastError();
}
hipError_t launch_step_cell(const void* Acat, const void* Wcell, const float* bias, const float* h_in, const float* c_in, float* h_out,
                            float* c_out, void* y, long ldy, float* cs, const int* lens, unsigned* status, int B, int n, int Kc, int ndir, hipStream_t s) {
  SkinnyArgs a = {};
  const int Np = 128 * cdiv(n, 32);
  a.A = (const char*)Acat; a.B = (const char*)Wcell; a.bias = bias;
  a.M = B; a.N = Np; a.K = Kc; a.lda = Kc; a.ldb = Kc;
  a.sAz = (long)B * Kc; a.sBz = (long)Np * Kc; a.nz = ndir;
  a.cell = 1; a.n = n; a.h_in = h_in; a.c_in = c_in; a.h_out = h_out; a.c_out = c_out; a.y = (uint16_t*)y; a.ldy = ldy; a.cs = cs; a.lens = lens; a.status = status;
  return launch(a, s);
}

}  // namespace lstm
