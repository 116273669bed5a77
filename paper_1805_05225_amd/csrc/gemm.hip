// Hoisted matrix products of the LSTM layer on the gfx950 matrix cores.
//
// Everything that does not depend on the recurrent state is taken out of the time loop
// (paper Sec. 3 and Sec. 7: computation is moved out of the recurrent loop) and done here as
// one large product per layer:
//   forward   Zx  = X   W_x + b        (A k-contiguous, B n-contiguous)
//   backward  dX  = DZ  W_x^T          (A k-contiguous, B k-contiguous, summed over directions)
//             dW_x = X^T  DZ           (A m-contiguous, B n-contiguous, K = all frames, masked)
//             dW_h = Hprev^T DZ        (same shape of problem)
//
// One kernel template covers the four layout combinations.  A 128x128 output tile is computed
// by 256 threads = 4 wavefronts (2x2), each owning a 64x64 sub-tile as 2x2 MFMA 32x32 blocks.
// Operand tiles are staged through LDS in k-contiguous rows of 128 bytes (+16 bytes padding, so
// 16-byte fragment reads of 16 consecutive rows fall into distinct banks).  Operands that are
// stored with m / n contiguous are transposed in registers on their way into LDS.  Global loads
// for tile i+1 are issued before the MFMAs of tile i (register staging, two LDS buffers).
#include "common.h"
#include <algorithm>
#include <type_traits>

namespace lstm {
namespace {

constexpr int kBM = 128, kBN = 128;
constexpr int kRowBytes = 128;            // bytes of k per LDS row: 64 bf16 or 32 float
constexpr int kLdsStride = 144;           // row stride in LDS (bytes)
constexpr int kTileBytes = kBM * kLdsStride;
constexpr int kThreads = 256;

template <typename T> struct Mma;
template <> struct Mma<bf16_t> {
  __device__ static f32x16 run(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<float> {
  // a 16-byte chunk holds 4 k per lane group; MFMA e contracts k-pair {e (lanes 0-31), 4+e (lanes 32-63)}
  __device__ static f32x16 run(uint4 a, uint4 b, f32x16 c) {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

// ---- k-contiguous operand: rows of the tile are rows of memory -------------------------------
// 128 rows x 8 chunks of 16 bytes; thread handles chunks tid + 256*i, i = 0..3
// Rows lie anywhere: 16 bytes are read from any address that an element may have.  No load is predicated (behind a branch each would be waited for by itself; with
// element by element where rows are not whole 16 bytes, a stage of 279 x 1853 x 515 took 7 us): rows past the last read another, and what lies past K or
// the rows is cleared when the stage goes into LDS (settle: any look at what was loaded waits for it).  The chunk that K ends in is read so that it ends with K, and
// shifted down then (K is at least a chunk: short_kernel).
template <typename T>
__device__ __forceinline__ void fetch_kcontig(uint32_t (&st)[16], const char* base, long ld, int rows, int row0,
                                              int K, int k0, int tid, const int (&prow)[4]) {
  constexpr int ES = sizeof(T), EPC = 16 / ES;
  struct __attribute__((packed, aligned(ES))) Chunk { uint32_t w[4]; };
  const int kc = k0 / EPC + (tid & 7);                                   // (k0 is a multiple of EPC)
  const long k = min((long)kc * EPC, (long)K - EPC);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const Chunk c = *(const Chunk*)(base + ((long)prow[i] * ld + k) * ES);   // prow[i]: where the row lies in memory (past the last: the tile's first)
#pragma unroll
    for (int j = 0; j < 4; ++j) st[4 * i + j] = c.w[j];
  }
}
template <typename T>
__device__ __forceinline__ void settle_kcontig(uint32_t (&st)[16], int rows, int row0, int K, int k0, int tid) {
  constexpr int ES = sizeof(T), EPC = 16 / ES;
  const int whole = K / EPC, kc = k0 / EPC + (tid & 7);
  if (k0 + 8 * EPC > K) {                                     // the stage that K ends in
    const int gone = EPC - (K - whole * EPC);                             // elements of the cut chunk that are not its own, in front: 1 .. EPC (EPC: there is none)
    const int d = gone * ES / 4, half = ES == 2 ? gone & 1 : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t w[4] = {st[4 * i], st[4 * i + 1], st[4 * i + 2], st[4 * i + 3]};
      if (d & 1) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0u; }
      if (d & 2) { w[0] = w[2]; w[1] = w[3]; w[2] = 0u; w[3] = 0u; }
      if (half) {
        w[0] = (w[0] >> 16) | (w[1] << 16); w[1] = (w[1] >> 16) | (w[2] << 16);
        w[2] = (w[2] >> 16) | (w[3] << 16); w[3] >>= 16;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) st[4 * i + j] = kc < whole ? st[4 * i + j] : kc == whole && gone < EPC ? w[j] : 0u;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (row0 + ((tid + kThreads * i) >> 3) >= rows)
#pragma unroll
      for (int j = 0; j < 4; ++j) st[4 * i + j] = 0u;
}
__device__ __forceinline__ void commit_kcontig(const uint32_t (&st)[16], char* lds, int tid) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int c = tid + kThreads * i;
    *(uint4*)(lds + (c >> 3) * kLdsStride + (c & 7) * 16) = make_uint4(st[4 * i], st[4 * i + 1], st[4 * i + 2], st[4 * i + 3]);
  }
}

// ---- m-contiguous operand: rows of memory are k, the tile is transposed in registers ----------
// frame mask: row k of the K axis is frame (t = k / Bt, b = k % Bt), valid iff t < lens[b]
// bf16: micro-tile of 8 k x 2 m (eight 4-byte loads at any address), two micro-tiles per thread; nothing predicated, as above: k past K reads the last
// row, columns past the last the last two, and both are cleared afterwards
template <bool MASK>
__device__ __forceinline__ void fetch_mcontig_bf16(uint32_t (&st)[16], const char* base, long ld, int cols, int col0,
                                                   int K, int k0, int tid, const int* lens, int Bt, int T, const int* krows, uint32_t (&kept)[4]) {
  struct __attribute__((packed, aligned(2))) Pair { uint32_t w; };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int c = tid + kThreads * i;
    int m = col0 + 2 * (c & 63), kb = __builtin_amdgcn_readfirstlane(k0 + (c >> 6) * 8);   // (the same in every lane of a wavefront)
    // The frame mask is fetched independently of the data and applied afterwards, so the data loads
    // never wait for the seq_lens loads.
    uint32_t keep = 0xffu;
    if (MASK) {
      int ft = kb / Bt, fb = kb - ft * Bt;                  // frame (t, b) of row kb, advanced incrementally
      keep = 0u;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        if (kb + kk < K) { int L = lens[fb]; L = L < 0 ? 0 : (L > T ? T : L); keep |= (ft < L ? 1u : 0u) << kk; }
        if (++fb == Bt) { fb = 0; ++ft; }
      }
    }
    if (cols == 1) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int k = min(kb + kk, K - 1);
        st[8 * i + kk] = *(const uint16_t*)(base + (long)(krows ? krows[k] : k) * ld * 2);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int k = min(kb + kk, K - 1);                  // the same in every lane: a scalar look-up
        st[8 * i + kk] = ((const Pair*)(base + ((long)(krows ? krows[k] : k) * ld + min(m, cols - 2)) * 2))->w;
      }
    }
    kept[i] = keep;
  }
}
__device__ __forceinline__ void settle_mcontig_bf16(uint32_t (&st)[16], int cols, int col0, int K, int k0, int tid, const uint32_t (&kept)[4]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = tid + kThreads * i, m = col0 + 2 * (c & 63), kb = __builtin_amdgcn_readfirstlane(k0 + (c >> 6) * 8);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      uint32_t w = st[8 * i + kk];
      if (m + 1 == cols && cols > 1) w >>= 16;              // the last column alone
      st[8 * i + kk] = m < cols && kb + kk < K && ((kept[i] >> kk) & 1u) ? w : 0u;
    }
  }
}
__device__ __forceinline__ void commit_mcontig_bf16(const uint32_t (&st)[16], char* lds, int tid) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int c = tid + kThreads * i;
    int r = 2 * (c & 63), kc = c >> 6;
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t a = st[8 * i + 2 * j], b = st[8 * i + 2 * j + 1];
      lo[j] = (a & 0xffffu) | (b << 16);
      hi[j] = (a >> 16) | (b & 0xffff0000u);
    }
    *(uint4*)(lds + r * kLdsStride + kc * 16) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    *(uint4*)(lds + (r + 1) * kLdsStride + kc * 16) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  }
}
// float: micro-tile of 4 k x 1 m, four per thread
template <bool MASK>
__device__ __forceinline__ void fetch_mcontig_f32(uint32_t (&st)[16], const char* base, long ld, int cols, int col0,
                                                  int K, int k0, int tid, const int* lens, int Bt, int T, const int* krows, uint32_t (&kept)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int c = tid + kThreads * i;
    int m = col0 + (c & 127), kb = __builtin_amdgcn_readfirstlane(k0 + (c >> 7) * 4);     // (the same in every lane of a wavefront)
    uint32_t keep = 0xfu;
    if (MASK) {
      int ft = kb / Bt, fb = kb - ft * Bt;
      keep = 0u;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (kb + kk < K) { int L = lens[fb]; L = L < 0 ? 0 : (L > T ? T : L); keep |= (ft < L ? 1u : 0u) << kk; }
        if (++fb == Bt) { fb = 0; ++ft; }
      }
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int k = min(kb + kk, K - 1);                                     // (a scalar look-up)
      st[4 * i + kk] = *(const uint32_t*)(base + ((long)(krows ? krows[k] : k) * ld + min(m, cols - 1)) * 4);
    }
    kept[i] = keep;
  }
}
__device__ __forceinline__ void settle_mcontig_f32(uint32_t (&st)[16], int cols, int col0, int K, int k0, int tid, const uint32_t (&kept)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + kThreads * i, m = col0 + (c & 127), kb = __builtin_amdgcn_readfirstlane(k0 + (c >> 7) * 4);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      if (!(m < cols && kb + kk < K && ((kept[i] >> kk) & 1u))) st[4 * i + kk] = 0u;
  }
}
__device__ __forceinline__ void commit_mcontig_f32(const uint32_t (&st)[16], char* lds, int tid) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int c = tid + kThreads * i;
    *(uint4*)(lds + (c & 127) * kLdsStride + (c >> 7) * 16) = make_uint4(st[4 * i], st[4 * i + 1], st[4 * i + 2], st[4 * i + 3]);
  }
}

// A stage of one operand: K, rows (columns of a k-major one) in force; `mapped`: its k-rows are those of g.k_rows
template <typename T, bool KCONTIG, bool MASK>
struct Stager {
  static constexpr int EPT = kRowBytes / (int)sizeof(T);   // k per tile: 64 bf16 / 32 float
  uint32_t st[16], kept[4];
  __device__ __forceinline__ void fetch(const GemmArgs& g, const char* base, long ld, int rows, int K, int at, int k0, int tid, const int (&prow)[4], bool mapped) {
    const int* krows = mapped ? g.k_rows : nullptr;
    if constexpr (KCONTIG) fetch_kcontig<T>(st, base, ld, rows, at, K, k0, tid, prow);
    else if constexpr (sizeof(T) == 2) fetch_mcontig_bf16<MASK>(st, base, ld, rows, at, K, k0, tid, g.lens, g.Bt, g.T, krows, kept);
    else fetch_mcontig_f32<MASK>(st, base, ld, rows, at, K, k0, tid, g.lens, g.Bt, g.T, krows, kept);
  }
  __device__ __forceinline__ void commit(char* lds, int rows, int K, int at, int k0, int tid) {
    if constexpr (KCONTIG) { settle_kcontig<T>(st, rows, at, K, k0, tid); commit_kcontig(st, lds, tid); }
    else if constexpr (sizeof(T) == 2) { settle_mcontig_bf16(st, rows, at, K, k0, tid, kept); commit_mcontig_bf16(st, lds, tid); }
    else { settle_mcontig_f32(st, rows, at, K, k0, tid, kept); commit_mcontig_f32(st, lds, tid); }
  }
};

template <typename T, typename TC, bool AK, bool BK, bool MASK>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmArgs g) {
  using SA = Stager<T, AK, MASK>;
  using SB = Stager<T, BK, false>;
  constexpr int EPT = SA::EPT;
  __shared__ __attribute__((aligned(16))) char lds[4 * kTileBytes];   // A0 B0 A1 B1
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int r = lane & 31, gq = lane >> 5;

  // tile raster: bands of 8 tile-columns, row-major inside a band, so that the eight XCDs
  // (work-groups are dealt to them round-robin) each keep one B tile-column in their L2.
  const int tiles_m = (g.M + kBM - 1) / kBM, tiles_n = (g.N + kBN - 1) / kBN;
  int bid = blockIdx.x;
  const int band = bid / (8 * tiles_m);
  const int width = min(8, tiles_n - band * 8);
  const int rel = bid - band * 8 * tiles_m;
  const int tn = band * 8 + rel % width, tm = rel / width;
  const int m0 = tm * kBM, n0 = tn * kBN;
  const int z = blockIdx.y;
  // Row maps and device-side extents (the frames that are real, numbered on the device): logical row r of a k-contiguous A
  // and of C is row a_rows[r] / c_rows[r] in memory, M is cut down to *m_dev; with both operands m-contiguous, row k of
  // the K axis is row k_rows[k] of A and of B, K cut down to *k_dev.
  const int M = g.m_dev ? min(g.M, *g.m_dev) : g.M;
  const int K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  if (m0 >= M) return;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // where the rows this thread stages lie in memory (k-contiguous operands: the same rows in every stage)
  int arow[4], brow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ra = m0 + ((tid + kThreads * i) >> 3);
    arow[i] = ra < M ? ra : m0;
    if (AK && g.a_rows) arow[i] = g.a_rows[arow[i]];
    const int rb = n0 + ((tid + kThreads * i) >> 3);
    brow[i] = rb < g.N ? rb : n0;
  }
  const int ktiles = (K + EPT - 1) / EPT;
  const int total = ktiles * g.nseg;
  SA sa[2];                                                 // stages on their way from memory: two, or every stage is a round trip
  SB sb[2];
  auto fetch = [&](int it, int set) __attribute__((always_inline)) {
    int seg = it / ktiles, kt = it - seg * ktiles;
    const char* A = (const char*)g.A + (g.sAz * z + g.sAseg * seg) * (long)sizeof(T);
    const char* B = (const char*)g.B + (g.sBz * z + g.sBseg * seg) * (long)sizeof(T);
    sa[set].fetch(g, A, g.lda, M, K, m0, kt * EPT, tid, arow, !AK);
    sb[set].fetch(g, B, g.ldb, g.N, K, n0, kt * EPT, tid, brow, !AK && !BK);
  };
  auto commit = [&](int it, int set) __attribute__((always_inline)) {        // into LDS buffer `set`
    const int k0 = it % ktiles * EPT;
    sa[set].commit(lds + set * 2 * kTileBytes, M, K, m0, k0, tid);
    sb[set].commit(lds + set * 2 * kTileBytes + kTileBytes, g.N, K, n0, k0, tid);
  };
  // stage `it` is in LDS buffer it % 2, stage it + 1 in register set (it + 1) % 2
  auto stage = [&](int it, int cur) __attribute__((always_inline)) {
    if (it + 2 < total) fetch(it + 2, cur);
    const char* As = lds + cur * 2 * kTileBytes + (wm * 64 + r) * kLdsStride + gq * 16;
    const char* Bs = lds + cur * 2 * kTileBytes + kTileBytes + (wn * 64 + r) * kLdsStride + gq * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint4 a0 = *(const uint4*)(As + j * 32), a1 = *(const uint4*)(As + 32 * kLdsStride + j * 32);
      uint4 b0 = *(const uint4*)(Bs + j * 32), b1 = *(const uint4*)(Bs + 32 * kLdsStride + j * 32);
      acc[0][0] = Mma<T>::run(a0, b0, acc[0][0]);
      acc[0][1] = Mma<T>::run(a0, b1, acc[0][1]);
      acc[1][0] = Mma<T>::run(a1, b0, acc[1][0]);
      acc[1][1] = Mma<T>::run(a1, b1, acc[1][1]);
    }
    if (it + 1 < total) commit(it + 1, cur ^ 1);
    __syncthreads();
  };
  if (total > 0) {
    fetch(0, 0);
    if (total > 1) fetch(1, 1);
    commit(0, 0);
  }
  __syncthreads();
  for (int it = 0; it < total; it += 2) {
    stage(it, 0);
    if (it + 1 < total) stage(it + 1, 1);
  }

  // epilogue: lane holds column (lane % 32), rows 8*(v/4) + 4*(lane/32) + v%4 of each 32x32 block.  Row map and, for an accumulating product, C are
  // read for a whole block before the first store: a read behind a store waits for it (element by element the epilogue alone took 15 us).
  TC* C = (TC*)g.C + g.sCz * z;
  const float* bias = g.bias ? g.bias + g.sbiasz * z : nullptr;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row0 = m0 + wm * 64 + i * 32 + 4 * gq;
    int crow[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) crow[v] = min(row0 + 8 * (v >> 2) + (v & 3), M - 1);
    if (g.c_rows) {
#pragma unroll
      for (int v = 0; v < 16; ++v) crow[v] = g.c_rows[crow[v]];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn * 64 + j * 32 + r, ccol = min(col, g.N - 1);
      const float bv = bias ? bias[ccol] : 0.f;
      float val[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) val[v] = acc[i][j][v] + bv;
      if constexpr (sizeof(TC) == 4) {
        if (g.accumulate) {
          float old[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) old[v] = ((const float*)C)[(long)crow[v] * g.ldc + ccol];
#pragma unroll
          for (int v = 0; v < 16; ++v) val[v] += old[v];
        }
      }
      if (col >= g.N) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (row0 + 8 * (v >> 2) + (v & 3) < M) Store<typename std::conditional<sizeof(TC) == 4, float, bf16_t>::type>::store(C, (long)crow[v] * g.ldc + col, val[v]);
    }
  }
}

// k-contiguous operands of less than a chunk, K < 16 / sizeof(T): little more than storing C.  Small results are bound by the chain from the loads to the store: a thread per element of C, with
// its operands from memory.
template <typename T, typename TC>
__global__ __launch_bounds__(256) void short_element_kernel(GemmArgs g) {
  const int idx = blockIdx.x * 256 + threadIdx.x, m = idx / g.N, n = idx - m * g.N, z = blockIdx.y;      // (at most 2^21 of them)
  if (m >= (g.m_dev ? min(g.M, *g.m_dev) : g.M)) return;
  const int K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  float v = g.bias ? g.bias[g.sbiasz * z + n] : 0.f;
  for (int seg = 0; seg < g.nseg; ++seg)
    for (int k = 0; k < K; ++k) {
      const long b_at = g.b_kcontig ? (long)n * g.ldb + k : (long)k * g.ldb + n;
      v += Store<T>::load(g.A, g.sAz * z + g.sAseg * seg + (long)(g.a_rows ? g.a_rows[m] : m) * g.lda + k) * Store<T>::load(g.B, g.sBz * z + g.sBseg * seg + b_at);
    }
  const long off = g.sCz * z + (long)(g.c_rows ? g.c_rows[m] : m) * g.ldc + n;
  if (g.accumulate) v += Store<TC>::load(g.C, off);
  Store<TC>::store(g.C, off, v);
}
// Larger ones: a thread owns a column and R rows of a tile of `cols` columns: its column of B in registers, the tile's rows of A in LDS, from where a wavefront's rows are read by all lanes at
// once.  us, gemm_kernel / a thread per element / so: 4096 x 4096 into float, K = 4 33.5 / 59.5 / 30.2, K = 7 37.5 / 81 / 31; 768 x 20000 33.8 / 53.9 / 28.1 and 38.3 / 71.6 / 29.0.
// The line lies where the two take the same: a million elements (310 x 2983 x 3 5.4 / 4.8, 1803 x 516 x 7 7.3 / 6.6, 13986 x 76 x 2 5.4 / 7.9, 106199 x 5 x 4 4.6 / 7.2), twice that with at most
// three k (90551 x 23 x 1 8.0 / 8.2, 1057 x 1405 x 3 7.4 / 6.9) or less than sixteen columns, the narrowest tile (280032 x 5 x 7 11.6 / 16.6).
bool short_by_element(const GemmArgs& g) { return (long)g.M * g.N * g.nz <= 1L << (g.K <= 3 || g.N < 16 ? 21 : 20); }
constexpr int kShortGrid = 1 << 16;
template <typename T, typename TC, int R>
__global__ __launch_bounds__(256) void short_kernel(GemmArgs g, int cols, long tiles_n, long tiles) {
  constexpr int E = 16 / (int)sizeof(T);
  __shared__ __attribute__((aligned(16))) float a[256][E];                     // (at most 16 rows a thread, and at least 16 columns: 256 rows)
  const int tid = threadIdx.x, z = blockIdx.y, c = tid & (cols - 1), r0 = tid / cols, par = 256 / cols, rows = R * par;
  const int M = g.m_dev ? min(g.M, *g.m_dev) : g.M, K = g.k_dev ? min(g.K, *g.k_dev) : g.K;
  for (long t = blockIdx.x; t < tiles; t += gridDim.x) {
    const long tm = t / tiles_n, m0 = tm * rows, n = (t - tm * tiles_n) * cols + c;
    if (m0 >= M) return;
    float acc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = g.bias && n < g.N ? g.bias[g.sbiasz * z + n] : 0.f;
    for (int seg = 0; seg < g.nseg; ++seg) {
      __syncthreads();                                                        // (what is in LDS has been read)
      for (int i = tid; i < rows * E; i += 256) {
        const long m = m0 + i / E;
        const int k = i % E;
        a[i / E][k] = m < M && k < K ? Store<T>::load(g.A, g.sAz * z + g.sAseg * seg + (g.a_rows ? g.a_rows[m] : m) * g.lda + k) : 0.f;
      }
      float b[E];
#pragma unroll
      for (int k = 0; k < E; ++k)
        b[k] = n < g.N && k < K ? Store<T>::load(g.B, g.sBz * z + g.sBseg * seg + (g.b_kcontig ? n * g.ldb + k : k * g.ldb + n)) : 0.f;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < E; ++k) acc[i] += a[i * par + r0][k] * b[k];
    }
    if (n >= g.N) continue;
    long off[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const long m = std::min(m0 + i * par + r0, M - 1L);
      off[i] = g.sCz * z + (g.c_rows ? g.c_rows[m] : m) * g.ldc + n;
    }
    if (g.accumulate) {
#pragma unroll
      for (int i = 0; i < R; ++i) acc[i] += Store<TC>::load(g.C, off[i]);
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (m0 + i * par + r0 < M) Store<TC>::store(g.C, off[i], acc[i]);
  }
}
template <typename T, typename TC>
hipError_t launch_short(const GemmArgs& g, hipStream_t s) {
  if (short_by_element(g)) {
    hipLaunchKernelGGL((short_element_kernel<T, TC>), dim3(cdiv((long)g.M * g.N, 256), g.nz), dim3(256), 0, s, g);
    return hipGetLastError();
  }
  int cols = 16;
  while (cols < 256 && cols < g.N) cols *= 2;
  const int par = 256 / cols;
  const int r = g.M >= 16 * par ? 16 : g.M >= 4 * par ? 4 : 1;                                                // rows a thread
  const long tiles_n = ((long)g.N + cols - 1) / cols, tiles = tiles_n * (((long)g.M + r * par - 1) / (r * par));
  const dim3 grid((unsigned)std::min(tiles, (long)kShortGrid), g.nz);
  if (r == 16) hipLaunchKernelGGL((short_kernel<T, TC, 16>), grid, dim3(256), 0, s, g, cols, tiles_n, tiles);
  else if (r == 4) hipLaunchKernelGGL((short_kernel<T, TC, 4>), grid, dim3(256), 0, s, g, cols, tiles_n, tiles);
  else hipLaunchKernelGGL((short_kernel<T, TC, 1>), grid, dim3(256), 0, s, g, cols, tiles_n, tiles);
  return hipGetLastError();
}

template <typename T, typename TC>
hipError_t dispatch(const GemmArgs& g, hipStream_t s) {
  if (g.a_kcontig && g.K < 16 / (int)sizeof(T)) return launch_short<T, TC>(g, s);
  const int tiles_m = (g.M + kBM - 1) / kBM, tiles_n = (g.N + kBN - 1) / kBN;
  dim3 grid(tiles_m * tiles_n, g.nz), block(kThreads);
  if (g.a_kcontig && !g.b_kcontig) hipLaunchKernelGGL((gemm_kernel<T, TC, true, false, false>), grid, block, 0, s, g);
  else if (g.a_kcontig && g.b_kcontig) hipLaunchKernelGGL((gemm_kernel<T, TC, true, true, false>), grid, block, 0, s, g);
  else if (!g.a_kcontig && !g.b_kcontig && g.lens) hipLaunchKernelGGL((gemm_kernel<T, TC, false, false, true>), grid, block, 0, s, g);
  else if (!g.a_kcontig && !g.b_kcontig) hipLaunchKernelGGL((gemm_kernel<T, TC, false, false, false>), grid, block, 0, s, g);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// A handful of columns in bfloat16 and little K, rows or K of whole 8 bytes but not 16: the 128 x 128 tiles of gemm_tile.hip store a row's few bytes at a time and take as long as the
// kernel here takes for two stages (us, there / here: 6604 x 4 x 16 11.9 / 8.8, 1684 x 16 x 12 12.1 / 9.1, 2004 x 8 x 80 12.4 / 10.2; in float 8 / 9, and from 36 columns or 100 k on there).
// Less than a tile of rows is faster there (m-contiguous 28 x 12 x 20 5.7 / 7.0, 80 x 4 x 20 7.8 / 9.5).  The kernel here knows no padding of K and no ranges.
bool narrow_result(const GemmArgs& g) {
  const bool whole = ((g.lda | g.ldb | (g.a_kcontig ? g.K : 0)) & 7) == 0 && (((uintptr_t)g.A | (uintptr_t)g.B) & 15) == 0;
  return g.in_bf16 && g.out_bf16 && !whole && !g.k_phys_rows && !g.parts && g.M > kBM && g.N <= 32 && g.K < (g.b_kcontig ? 100 : 72);
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nz <= 0) return hipSuccess;
  if (!gemm_skinny_ok(g) && few_any_ok(g)) return launch_few_any(g, s);
  if (g.M > 64 && g.M <= kSkinnyMaxRows && g.a_kcontig && g.b_kcontig && g.nz == 1 && g.nseg == 1 && !g.parts && !g.a_rows && !g.c_rows && !g.m_dev && gemm_tile_ok(g) && gemm_nt_ok(g)) {
    const FewRoute r = few_rows_route(g.M, g.N, g.K);
    if (r != FewRoute::kHere) return r == FewRoute::kTile ? launch_gemm_tile(g, s) : launch_gemm_nt(g, s);
  }
  if (gemm_skinny_ok(g)) return launch_gemm_skinny(g, s);
  if (narrow_result(g)) return dispatch<bf16_t, bf16_t>(g, s);
  if (gemm_nn_ok(g) && (gemm_nn_pays(g) || !gemm_tile_ok(g))) return launch_gemm_nt(g, s);
  if (gemm_tile_ok(g) && (gemm_tile_small(g.M, g.N, g.nz) || (g.a_kcontig && !g.b_kcontig))) return launch_gemm_tile(g, s);
  if (gemm_nt_ok(g)) return launch_gemm_nt(g, s);
  if (gemm_tn_ok(g)) return launch_gemm_tn(g, s);
  if (gemm_float_ok(g)) return launch_gemm_float(g, s);
  if (g.in_bf16) {
    if (g.out_bf16) return dispatch<bf16_t, bf16_t>(g, s);
    return dispatch<bf16_t, float>(g, s);
  }
  if (g.out_bf16) return hipErrorInvalidValue;
  return dispatch<float, float>(g, s);
}

}  // namespace lstm
