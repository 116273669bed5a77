// Products with a handful of rows: the decoder step of one sentence (beam 12: 12 rows) or of a few.
//
//     C[M,N] = A[M,K] B[N,K]^T (+ bias, max(0, .)), or the LSTM cell of the stepped decoder in the epilogue
//
// With M up to a few dozen the product is a read of B: 29 MB of packed cell weights at n_in = 2620, n = 1000 against
// 0.3 GFLOP at 12 rows, i.e. 6 us at the rate a large copy reaches.  The tiles of gemm_skinny.hip (96 rows x 128 columns)
// put such a product on 32 compute units, each of which pulls its 0.9 MB through a pipeline of 64-wide stages: 31 us.
// Here a work-group owns `ct` <= 16 columns (for the cell: the four gates of four units) and up to sixteen wavefronts share its K,
// so that N = 4000 gives 250 work-groups and N = 1000 still does (ct = 4; the MFMA's other columns repeat them, the matrix
// cores have nothing else to do).  Operands go from memory straight into MFMA fragments - nothing is shared between
// wavefronts, so there is nothing to stage - with everything a wavefront needs of a small K in flight at once; the
// wavefronts' sums meet in LDS.  Rows come in blocks of 16 MT (grid y): B is read once per block.
//
// FRAG: both operands lie in memory in fragment order, [tile of 16 rows / columns][chunk of 32 k][lane] x 16 bytes (packed that
// way once per search for the weights, by the concatenation for A): a wavefront's load is 1 KiB in a row.  Otherwise they are
// row-major and k-contiguous, rows 16-byte aligned; neighbouring lanes then sit in different rows, each group of four
// touches four cache lines, and the load path takes four times as long - which is why the decoder's two large products
// are packed.  Both bfloat16, K a multiple of 8.
//
// ANY: rows of any length that begin at any element (K no multiple of 8, so rows begin anywhere): 16 bytes are read at any element.  The other kernels that take such rows are
// the 128 x 128 tiles and the generic kernel, a few work-groups that walk K one stage after the other: K = 1003, N = 1000, 4 rows 20.4 us, here 6.0.  A load that begins inside a
// word costs the load path about three, so odd K pays for fewer rows and columns than even (few_any_ok).
#include "recurrent_dev.h"
#include "gemm_skinny.h"

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices
constexpr unsigned kParked = 0x7ffffff0u;

__device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Pieces of up to three matrices side by side, [x0 | x1 | x2]: piece i covers columns k_i .. k_i + len_i - 1 of the result, whatever
// lies between is zero; x2 may be float (rounded where it is read) and NULL (zeros).
struct ConcatArgs {
  const uint16_t* x0; const uint16_t* x1; const void* x2;
  long ld0, ld1, ld2;
  int k0, len0, k1, len1, k2, len2;
  int B, nkc; long s2;                   // rows; chunks of 32 columns; elements between the directions' x2
  int cut[4];                            // groups of eight columns in which a piece begins or ends (-1: none)
  void find_cuts() {
    int have = 0;
    for (int e : {k0 + len0, k1 + len1, k2, k2 + len2}) {
      bool known = e % 8 == 0;
      for (int i = 0; i < have; ++i) known |= cut[i] == e / 8;
      if (!known) cut[have++] = e / 8;
    }
    while (have < 4) cut[have++] = -1;
  }
};
typedef uint4 __attribute__((aligned(2))) uint4_u;
typedef float4 __attribute__((aligned(4))) float4_u;
__device__ __forceinline__ uint4 frag_pack(const uint16_t (&v)[8]) {
  return make_uint4(v[0] | ((unsigned)v[1] << 16), v[2] | ((unsigned)v[3] << 16), v[4] | ((unsigned)v[5] << 16), v[6] | ((unsigned)v[7] << 16));
}
// eight floats rounded to bfloat16 (to nearest even)
__device__ __forceinline__ uint4 frag_pack(const float4& lo, const float4& hi) {
  typedef __attribute__((ext_vector_type(8))) float f32x8;
  return __builtin_bit_cast(uint4, __builtin_convertvector((f32x8){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}, bf16x8));
}
// columns k .. k + 7 of a row, one by one: where a piece begins or ends inside them
template <bool F32>
__device__ __forceinline__ uint4 concat_slow(const ConcatArgs& a, int z, int row, int k) {
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int c = k + e;
    v[e] = 0;
    if (c >= a.k0 && c < a.k0 + a.len0) v[e] = a.x0[row * a.ld0 + c - a.k0];
    else if (c >= a.k1 && c < a.k1 + a.len1) v[e] = a.x1[row * a.ld1 + c - a.k1];
    else if (a.x2 && c >= a.k2 && c < a.k2 + a.len2)
      v[e] = F32 ? f2bf_bits(((const float*)a.x2)[a.s2 * z + row * a.ld2 + c - a.k2]) : ((const uint16_t*)a.x2)[row * a.ld2 + c - a.k2];
  }
  return frag_pack(v);
}

// Sums of the wavefronts' shares, red[wavefront][row tile][row][column], and what is done with them.
template <int MT, int NW, bool CELL>
__device__ __forceinline__ void few_epilogue(const SkinnyArgs& g, int ct, const float (&red)[NW][MT][16][17]) {
  const int tid = threadIdx.x, z = blockIdx.z, m0 = blockIdx.y * (16 * MT), n0 = blockIdx.x * ct;
  if constexpr (CELL) {
    if (tid == 0 && (blockIdx.x | blockIdx.y | blockIdx.z) == 0) *g.status = 0u;
    // thread -> (row, unit of four)
    for (int idx = tid; idx < MT * 64; idx += 64 * NW) {
      const int u = idx & 3, row = idx >> 2, b = m0 + row, j = blockIdx.x * 4 + u, n = g.n;
      if (b >= g.M || j >= n) continue;
      const long si = ((long)z * g.M + b) * n + j;
      const bool valid = clamp_len(g.lens, b, 1) > 0;
      float c = g.c_in ? g.c_in[si] : 0.f, h = 0.f;
      if (valid) {
        float zh[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float s = g.bias ? g.bias[(long)z * 4 * n + q * n + j] : 0.f;
#pragma unroll
          for (int w = 0; w < NW; ++w) s += red[w][row >> 4][row & 15][4 * q + u];
          zh[q] = s;
        }
        const float zx[4] = {0.f, 0.f, 0.f, 0.f};
        const CellOut o = lstm_cell(zh, zx, c);
        c = o.c; h = o.h;
      }
      g.y[(long)b * g.ldy + (long)z * n + j] = f2bf_bits(h);
      if (g.cs) g.cs[si] = c;
      if (g.c_out) g.c_out[si] = c;
      if (g.h_out) g.h_out[si] = valid ? h : (g.h_in ? g.h_in[si] : 0.f);
    }
  } else {
    for (int idx = tid; idx < MT * 256; idx += 64 * NW) {
      const int cc = idx & 15, row = idx >> 4, m = m0 + row, c = n0 + cc;
      if (cc >= ct || m >= g.M || c >= g.N) continue;
      float s = g.bias ? g.bias[g.sbiasz * z + c] : 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[w][row >> 4][row & 15][cc];
      if (g.relu) s = s > 0.f ? s : 0.f;
      const long off = g.sCz * z + (long)m * g.ldc + c;
      if (g.out_bf16) ((uint16_t*)g.C)[off] = f2bf_bits(s);
      else ((float*)g.C)[off] = s;
    }
  }
}

// MT row tiles of 16 per work-group, NW wavefronts, U k-chunks (of 32) per wavefront in a batch; with DB the next batch's loads
// are in flight while a batch is multiplied.
template <int MT, int NW, int U, bool DB, bool FRAG, bool CELL, bool ANY>
__global__ __launch_bounds__(64 * NW) void few_kernel(SkinnyArgs g, int ct) {
  static_assert(U % 2 == 0, "chunks come in pairs: 128 bytes of a row");
  __shared__ float red[NW][MT][16][17];                        // [wavefront][row tile][row][column]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, gk = lane >> 4;
  const int z = blockIdx.z, m0 = blockIdx.y * (16 * MT), n0 = blockIdx.x * ct;
  const int K = g.K, npair = (K + 63) / 64;                    // pairs of chunks: 64 k

  // Columns past ct repeat others: quads of lanes stay on the same lines.  Rows past M: the last one again (row-major), or whatever
  // the packed rows hold there; both end in output rows that are not stored.
  const int col = r16 & (ct - 1);
  const int nkc = (K + 31) / 32;
  // ANY: a lane's eight k that K ends in or in front of are K's last eight, and masks leave of them what no other lane has; its lowest half word is element 8 - K % 8.
  u32x4 tail;
#pragma unroll
  for (int e = 0; e < 4; ++e) tail[e] = (2 * e >= 8 - (K & 7) ? 0xffffu : 0u) | (2 * e + 1 >= 8 - (K & 7) ? 0xffff0000u : 0u);
  const long a_bytes = FRAG ? (long)((g.M + 15) / 16) * nkc * 1024 : (long)g.M * g.lda * 2;
  const long b_bytes = FRAG ? (long)((CELL ? (g.n + 3) / 4 : (g.N + 15) / 16)) * nkc * 1024 : (long)g.N * g.ldb * 2;
  const auto rec = [](long bytes) { return (int)(bytes > 0x7fffff00L ? 0x7fffff00L : bytes); };
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)(g.A + g.sAz * z * 2), 0, rec(a_bytes), kBufFlags);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)(g.B + g.sBz * z * 2), 0, rec(b_bytes), kBufFlags);
  constexpr unsigned kChunk = FRAG ? 1024u : 64u;              // bytes from one chunk of a lane's row to the next
  unsigned ao[MT], bo;
  if constexpr (FRAG) {
    bo = (unsigned)((long)(CELL ? (int)blockIdx.x : n0 >> 4) * nkc * 1024) + (unsigned)(gk * 16 + (n0 & 15) + col) * 16u;
#pragma unroll
    for (int i = 0; i < MT; ++i) ao[i] = (unsigned)((long)min((m0 >> 4) + i, (g.M - 1) >> 4) * nkc * 1024) + (unsigned)lane * 16u;
  } else {
    bo = (unsigned)((long)min(n0 + col, g.N - 1) * g.ldb * 2) + (ANY ? 0u : gk * 16u);
#pragma unroll
    for (int i = 0; i < MT; ++i) ao[i] = (unsigned)((long)min(m0 + 16 * i + r16, g.M - 1) * g.lda * 2) + (ANY ? 0u : gk * 16u);
  }

  const char *pa = g.A + g.sAz * z * 2, *pb = g.B + g.sBz * z * 2;

  f32x4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // every work-group reads all of A: those of an XCD start at different places, so that they do not ask its L2 for the same
  // lines at the same time
  const int rot = (int)(((long)((blockIdx.x >> 3) & 31) * npair) >> 5);
  struct Batch { u32x4 a[U][MT], b[U]; int k[ANY ? U : 1]; };
  // Chunk j of a batch that starts at pair p: pair p + NW (j / 2), half j % 2.  A chunk past K arrives as zeros (both operands:
  // the other one may hold anything there).
  auto load = [&](Batch& x, int p) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int q = p + NW * (j >> 1), kp = q + rot;
      const int kc = q < npair ? 2 * (kp < npair ? kp : kp - npair) + (j & 1) : 0x1000000;
      if constexpr (ANY) {
        x.k[j] = kc * 32 + gk * 8;
        const unsigned col = (unsigned)min(x.k[j], K - 8) * 2u;
        x.b[j] = __builtin_bit_cast(u32x4, *(const uint4_u*)(pb + (bo + col)));
#pragma unroll
        for (int i = 0; i < MT; ++i) x.a[j][i] = __builtin_bit_cast(u32x4, *(const uint4_u*)(pa + (ao[i] + col)));
        continue;
      }
      const bool in = kc * 32 + gk * 8 < K;
      x.b[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, in ? bo + (unsigned)kc * kChunk : kParked, 0, 0);
#pragma unroll
      for (int i = 0; i < MT; ++i) x.a[j][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, in ? ao[i] + (unsigned)kc * kChunk : kParked, 0, 0);
    }
  };
  auto multiply = [&](const Batch& x) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      u32x4 keep = {~0u, ~0u, ~0u, ~0u};                       // (of both operands: what a row holds twice may be infinite)
      if constexpr (ANY) {
#pragma unroll
        for (int e = 0; e < 4; ++e) keep[e] = x.k[j] + 8 <= K ? ~0u : x.k[j] < K ? tail[e] : 0u;
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) acc[i] = ANY ? mma16(x.a[j][i] & keep, x.b[j] & keep, acc[i]) : mma16(x.a[j][i], x.b[j], acc[i]);
    }
  };
  constexpr int kAdvance = NW * U / 2;                         // pairs per batch of all wavefronts
  if constexpr (DB) {
    Batch x, y;
    int p = wave;
    if (p < npair) {
      load(x, p);
      for (;;) {
        if (p + kAdvance >= npair) { multiply(x); break; }
        load(y, p + kAdvance);
        multiply(x);
        p += kAdvance;
        if (p + kAdvance >= npair) { multiply(y); break; }
        load(x, p + kAdvance);
        multiply(y);
        p += kAdvance;
      }
    }
  } else {
    Batch x;
    for (int p = wave; p < npair; p += kAdvance) {
      load(x, p);
      __builtin_amdgcn_sched_barrier(0);                       // (all of them first: left alone the compiler keeps half in flight)
      multiply(x);
    }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][i][4 * gk + v][r16] = acc[i][v];
  __syncthreads();

  few_epilogue<MT, NW, CELL>(g, ct, red);
}

// The same for at most 16 rows with A taken from where its pieces lie, [x0 | x1 | x2]: no concatenation pass, whose launch
// costs as much as half of this kernel (12 rows, K = 3624: concatenation 4.1 us + product 8.0).  A wavefront reads a chunk with four
// neighbouring lanes per row (64 bytes in a row), turns it into fragment order through 1 KiB of LDS of its own - LDS
// operations of a wavefront happen in order, so nothing has to be waited for - and the weights, asked for first, arrive
// behind all of that.  B in fragment order, at most 16 * U * 32 values of k.
// Every work-group reads all of the pieces while others already store: outputs must not share a byte with them (a step in place,
// hT = h0, takes the concatenation).
template <int U, bool F32, bool CELL>
__global__ __launch_bounds__(1024) void few_gather_kernel(SkinnyArgs g, ConcatArgs ca, int ct) {
  constexpr int NW = 16, kHalf = U / 2;
  __shared__ float red[NW][1][16][17];
  __shared__ uint4 turn[NW][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, gk = lane >> 4, z = blockIdx.z, n0 = blockIdx.x * ct;
  const int nkc = ca.nkc, npair = (nkc + 1) / 2;
  const long b_bytes = (long)(CELL ? (g.n + 3) / 4 : (g.N + 15) / 16) * nkc * 1024;
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void*)(g.B + g.sBz * z * 2), 0, (int)(b_bytes > 0x7fffff00L ? 0x7fffff00L : b_bytes), kBufFlags);
  const unsigned bo = (unsigned)((long)(CELL ? (int)blockIdx.x : n0 >> 4) * nkc * 1024) + (unsigned)(gk * 16 + (n0 & 15) + (r16 & (ct - 1))) * 16u;
  const int rot = (int)(((long)((blockIdx.x >> 3) & 31) * npair) >> 5);      // (see few_kernel)
  auto chunk = [&](int j) __attribute__((always_inline)) {     // chunk j of this wavefront; nkc or more: none
    const int q = wave + NW * (j >> 1), kp = q + rot;
    return q < npair ? 2 * (kp < npair ? kp : kp - npair) + (j & 1) : 0x1000000;
  };
  // Every lane loads twice 16 bytes: the two halves of eight floats, or the same eight bfloat16, or (nothing to read there, or a piece
  // begins or ends inside the eight) the weights' first bytes, to be replaced by zeros.  A goes out in front of the weights:
  // loads return in order, and A, out of L2, is turned while the weights are on their way.
  const int row = lane >> 2, arow = min(row, g.M - 1);         // rows past M: the last one again
  uint4 lo[U], hi[U];
  unsigned as_float = 0u, as_zero = 0u;                        // a bit per chunk
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int k = chunk(j) * 32 + (lane & 3) * 8;
    const bool in0 = k >= ca.k0 && k + 8 <= ca.k0 + ca.len0, in1 = k >= ca.k1 && k + 8 <= ca.k1 + ca.len1;
    const bool in2 = ca.x2 && k >= ca.k2 && k + 8 <= ca.k2 + ca.len2;
    const char* p0 = (const char*)(ca.x0 + arow * ca.ld0 + (k - ca.k0));
    const char* p1 = (const char*)(ca.x1 + arow * ca.ld1 + (k - ca.k1));
    const char* p2 = F32 ? (const char*)((const float*)ca.x2 + ca.s2 * z + arow * ca.ld2 + (k - ca.k2))
                         : (const char*)((const uint16_t*)ca.x2 + arow * ca.ld2 + (k - ca.k2));
    const char* p = in0 ? p0 : in1 ? p1 : in2 ? p2 : (const char*)g.B;
    lo[j] = *(const uint4_u*)p;
    if (F32) hi[j] = *(const uint4_u*)(p + (in2 ? 16 : 0));
    as_float |= (F32 && in2 ? 1u : 0u) << j;
    as_zero |= (in0 || in1 || in2 ? 0u : 1u) << j;
  }
  __builtin_amdgcn_sched_barrier(0);
  u32x4 b[U];
#pragma unroll
  for (int j = 0; j < U; ++j) b[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, chunk(j) < nkc ? bo + (unsigned)chunk(j) * 1024u : kParked, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc[1] = {(f32x4){0.f, 0.f, 0.f, 0.f}};
  u32x4 a[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    uint4 v = lo[j];
    if (F32 && ((as_float >> j) & 1u)) v = frag_pack(__builtin_bit_cast(float4, lo[j]), __builtin_bit_cast(float4, hi[j]));
    if ((as_zero >> j) & 1u) v = make_uint4(0, 0, 0, 0);
    turn[wave][(lane & 3) * 16 + row] = v;
    asm volatile("" ::: "memory");
    a[j] = __builtin_bit_cast(u32x4, turn[wave][lane]);
    asm volatile("" ::: "memory");
  }
#pragma unroll
  for (int j = 0; j < U; ++j) acc[0] = mma16(a[j], b[j], acc[0]);
  // groups of eight k in which a piece begins or ends: a product of their own, the rest of the chunk zero
  if (wave < 4 && ca.cut[wave] >= 0) {
    const int g8 = ca.cut[wave];
    uint4 v = make_uint4(0, 0, 0, 0);
    if (gk == (g8 & 3)) v = concat_slow<F32>(ca, z, min(r16, g.M - 1), g8 * 8);
    const u32x4 bx = __builtin_amdgcn_raw_buffer_load_b128(rb, bo + (unsigned)(g8 >> 2) * 1024u, 0, 0);
    acc[0] = mma16(__builtin_bit_cast(u32x4, v), bx, acc[0]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][0][4 * gk + v][r16] = acc[0][v];
  __syncthreads();
  few_epilogue<1, NW, CELL>(g, ct, red);
}

template <int MT, int NW, int U, bool DB, bool FRAG, bool CELL, bool ANY>
hipError_t launch_as(const SkinnyArgs& a, int ct, int tiles_n, hipStream_t s) {
  hipLaunchKernelGGL((few_kernel<MT, NW, U, DB, FRAG, CELL, ANY>), dim3(tiles_n, cdiv(a.M, 16 * MT), a.nz), dim3(64 * NW), 0, s, a, ct);
  return hipGetLastError();
}
// Four wavefronts, eight chunks each, hold K = 1024 in one batch; a longer K takes sixteen.
template <bool FRAG, bool CELL, bool ANY = false>
hipError_t launch_rows(const SkinnyArgs& a, int ct, int tiles_n, hipStream_t s) {
  const bool longk = a.K > 1024;
  if constexpr (ANY) {
    if (a.K <= 512) {
      if (a.M <= 16) return launch_as<1, 4, 4, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
      if (a.M <= 32) return launch_as<2, 4, 4, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
      return launch_as<4, 4, 4, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    }
    // (Two batches of four chunks of two row tiles, or of two of four, do not fit 128 registers beside the masks.  us, those with what spilled / these, the mean of 60 to 2400 columns: 20 and 32
    // rows, K = 1067 14.2 / 8.5, 1801 15.0 / 13.9, 2801 27.2 / 20.7, 4094 13.5 / 11.9; 50 to 200 rows, K = 1419 20.1 / 19.8, 2377 34.4 / 33.3, 4094 22.8 / 21.6.)
    if (a.M > 16 && longk) return a.M <= 32 ? launch_as<2, 16, 2, true, FRAG, CELL, ANY>(a, ct, tiles_n, s) : launch_as<4, 16, 2, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    if (longk) return a.K <= 2048 ? launch_as<1, 16, 4, false, FRAG, CELL, ANY>(a, ct, tiles_n, s) : launch_as<1, 16, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    if (a.M <= 16) return launch_as<1, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    if (a.M <= 32) return launch_as<2, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    return launch_as<4, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
  } else {
    if (a.M <= 16) return longk ? launch_as<1, 16, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s) : launch_as<1, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    if (a.M <= 32) return longk ? launch_as<2, 16, 4, true, FRAG, CELL, ANY>(a, ct, tiles_n, s) : launch_as<2, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
    return longk ? launch_as<4, 16, 2, true, FRAG, CELL, ANY>(a, ct, tiles_n, s) : launch_as<4, 4, 8, false, FRAG, CELL, ANY>(a, ct, tiles_n, s);
  }
}

// Weights of the stepped cell: tile t holds the gates of units 4 t .. 4 t + 3 (column 4 q + u), k runs over [x | 0 | h | 0].
// A work-group turns 64 k x 64 units through LDS, so that W is read along its columns.
__global__ __launch_bounds__(256) void pack_cell_frag_kernel(const uint16_t* Wx, const uint16_t* Wh, uint4* out, int n_in, int n_in_pad, int n, int nkc,
                                                             int ntile) {
  __shared__ uint16_t tile[64][66];                            // [k][unit]
  const int d = blockIdx.z >> 2, q = blockIdx.z & 3, k0 = blockIdx.x * 64, u0 = blockIdx.y * 64, N4 = 4 * n;
  Wx += (long)d * n_in * N4;
  Wh += (long)d * n * N4;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6, j = u0 + tx;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int k = k0 + ty + 4 * i;
    uint16_t v = 0;
    if (j < n) {
      if (k < n_in) v = Wx[(long)k * N4 + q * n + j];
      else if (k >= n_in_pad && k < n_in_pad + n) v = Wh[(long)(k - n_in_pad) * N4 + q * n + j];
    }
    tile[ty + 4 * i][tx] = v;
  }
  __syncthreads();
#pragma unroll
  for (int rep = 0; rep < 2; ++rep) {                          // 64 units x 8 groups of eight k
    const int idx = threadIdx.x + 256 * rep, u = idx & 63, g8 = idx >> 6, kc = k0 / 32 + (g8 >> 2), unit = u0 + u, t = unit >> 2;
    if (t >= ntile || kc >= nkc) continue;
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[g8 * 8 + e][u];
    out[(((long)d * ntile + t) * nkc + kc) * 64 + (g8 & 3) * 16 + q * 4 + (unit & 3)] = frag_pack(v);
  }
}

// W[R][K] twice from one read: rows padded with zeros to Kp columns (a multiple of 8), and in fragment order.  Threads run along the rows.
__global__ __launch_bounds__(256) void pack_rows_both_kernel(const uint16_t* W, uint4* rows, uint4* frag, int R, int K, int Kp, int nkc, long total) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int kk = (int)(idx % (nkc * 4)), k = kk * 8;           // total = rows of whole tiles x groups of eight columns
  const long row = idx / (nkc * 4);
  uint4 o = make_uint4(0, 0, 0, 0);
  if (row < R && k + 8 <= K) o = *(const uint4_u*)(W + row * K + k);
  else if (row < R) {
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = k + e < K ? W[row * K + k + e] : (uint16_t)0;
    o = frag_pack(v);
  }
  if (row < R && k < Kp) rows[(row * Kp + k) / 8] = o;
  frag[((row >> 4) * nkc + (kk >> 2)) * 64 + (kk & 3) * 16 + (row & 15)] = o;
}

// [x0 | x1 | x2] in fragment order (grid y: direction); the rows that fill up the last tile are zero
template <bool F32>
__global__ void concat_frag_kernel(ConcatArgs a, uint4* out, long total) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  // (a row's threads are neighbours: reads run along the rows)
  const int kk = (int)(idx % (a.nkc * 4)), row = (int)(idx / (a.nkc * 4)), k = kk * 8, z = blockIdx.y;
  const auto inside = [&](int b, int len) { return k >= b && k + 8 <= b + len; };
  uint4 o = make_uint4(0, 0, 0, 0);
  if (row < a.B) {
    if (inside(a.k0, a.len0)) o = *(const uint4_u*)(a.x0 + row * a.ld0 + (k - a.k0));
    else if (inside(a.k1, a.len1)) o = *(const uint4_u*)(a.x1 + row * a.ld1 + (k - a.k1));
    else if (inside(a.k2, a.len2) && a.x2) {
      if constexpr (F32) {
        const float* p = (const float*)a.x2 + a.s2 * z + row * a.ld2 + (k - a.k2);
        o = frag_pack(*(const float4_u*)p, *(const float4_u*)(p + 4));
      } else {
        o = *(const uint4_u*)((const uint16_t*)a.x2 + row * a.ld2 + (k - a.k2));
      }
    } else {
      o = concat_slow<F32>(a, z, row, k);
    }
  }
  const long tiles = (a.B + 15) / 16;
  out[((tiles * z + (row >> 4)) * a.nkc + (kk >> 2)) * 64 + (kk & 3) * 16 + (row & 15)] = o;
}

constexpr int kGatherU = 8;              // chunks per wavefront: K up to 4096
// columns per work-group: as many as still give most compute units one
int few_columns(int M, int N) {
  const long blocks = M <= 64 ? 1 : cdiv(M, 64);
  return blocks * cdiv(N, 16) >= 192 ? 16 : blocks * cdiv(N, 8) >= 192 ? 8 : 4;
}

}  // namespace

hipError_t launch_few(const SkinnyArgs& a, hipStream_t s) {
  const int ct = few_columns(a.M, a.N);
  return a.frag ? launch_rows<true, false>(a, ct, cdiv(a.N, ct), s) : launch_rows<false, false>(a, ct, cdiv(a.N, ct), s);
}

// columns of a work-group: as few as still give one round of compute units
static int any_columns(long M, long N, int nz) {
  const long blocks = (long)cdiv(M, 64) * nz;
  return blocks * cdiv(N, 4) <= 256 ? 4 : blocks * cdiv(N, 8) <= 256 ? 8 : 16;
}
// Both sides estimated from measurements (us; 2 to 1024 rows, 263 to 32000 columns, 24 lengths of K from 60 to 4050, 4060 products).  Here: rounds of work-groups times what
// a wavefront loads, twice or three times as much if every other row begins inside a word (K odd); the other kernels: hardly anything but K.  It has to look a fifth faster (for
// K > 1024, whose rounds vary more, two fifths): slower choices are then 26 of those products, by 8 % in the median, and what is left behind is 1.25 times this.
// us, before / here: K = 334, N = 1000 10.5 / 5.0 for up to 256 rows, 12.1 / 8.1 for 768; K = 1003 20.4 / 6.0 for 4 rows, 22.6 / 13.4 for 64; K = 1012 (rows of whole 8 bytes) 11.7 / 4.9 for 4, 14.6 /
// 6.3 for 128; K = 505, N = 2787 13.1 / 7 for 16; K = 803, N = 20000 18.4 / 17.7 for 4 and 20.7 / 51 for 64, which stay where they were.
bool few_any_ok(const GemmArgs& g) {
  const long lim = 0x7fffff00L;                                // operands are addressed with 32-bit byte offsets
  if (g.M > kSkinnyMaxRows || !g.in_bf16 || !g.a_kcontig || !g.b_kcontig || g.lens || g.nseg != 1 || g.a_rows || g.c_rows || g.m_dev || g.k_dev || g.accumulate || g.parts || g.K < 8 ||
      ((long)g.M * g.lda + g.K) * 2 > lim || ((long)g.N * g.ldb + g.K) * 2 > lim)
    return false;
  const long M = g.M, groups = (long)cdiv(M, 64) * g.nz * cdiv(g.N, any_columns(M, g.N, g.nz));
  const int waves = g.K <= 1024 ? 4 : 16, deep = g.K <= 512 ? 4 : g.K <= 1024 ? 8 : M <= 16 ? (g.K <= 2048 ? 4 : 8) : 2;
  const double loads = (groups > 512 ? groups / 256. : (double)cdiv(groups, 256)) * waves * deep * cdiv(cdiv(g.K, 32), waves * deep), rows = (M < 64 ? M : 64) / 16.;
  const bool odd = ((g.lda | g.ldb) & 1) || (((uintptr_t)g.A | (uintptr_t)g.B) & 3);
  const double here = odd ? std::max(5.2, 3.6 + loads * (0.068 + 0.052 * rows)) : std::max(5.2, 4.2 + loads * (0.020 + 0.0155 * rows));
  const double there = gemm_tile_ok(g) ? 5.8 + 0.006 * g.K + 0.03 * (M < 128 ? M : 128) : (odd ? 5.6 : 6.0) + 0.0145 * g.K;
  return (g.K > 1024 ? 1.4 : 1.2) * here < there;
}
hipError_t launch_few_any(const GemmArgs& g, hipStream_t s) {
  SkinnyArgs a = {};
  a.A = (const char*)g.A; a.B = (const char*)g.B; a.C = g.C; a.bias = g.bias;
  a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
  a.sAz = g.sAz; a.sBz = g.sBz; a.sCz = g.sCz; a.sbiasz = g.sbiasz; a.nz = g.nz;
  a.out_bf16 = g.out_bf16;
  const int ct = any_columns(a.M, a.N, a.nz);
  return launch_rows<false, false, true>(a, ct, cdiv(a.N, ct), s);
}

hipError_t launch_pack_cell_frag(const void* W_x, const void* W_h, void* out, int n_in, int n_in_pad, int n, int K, int ndir, hipStream_t s) {
  const int nkc = cdiv(K, 32), ntile = cdiv(n, 4);
  hipLaunchKernelGGL(pack_cell_frag_kernel, dim3(cdiv(nkc, 2), cdiv(4L * ntile, 64), 4 * ndir), dim3(256), 0, s, (const uint16_t*)W_x,
                     (const uint16_t*)W_h, (uint4*)out, n_in, n_in_pad, n, nkc, ntile);
  return hipGetLastError();
}
hipError_t launch_pack_rows_both(const void* W, void* rows, void* frag, int R, int K, int Kp, hipStream_t s) {
  const int nkc = cdiv(K, 32);
  const long total = (long)cdiv(R, 16) * 16 * nkc * 4;
  hipLaunchKernelGGL(pack_rows_both_kernel, dim3(cdiv(total, 256)), dim3(256), 0, s, (const uint16_t*)W, (uint4*)rows, (uint4*)frag, R, K, Kp, nkc, total);
  return hipGetLastError();
}

hipError_t launch_few_cell(const void* x, const float* h_in, void* A, const void* Wfrag, const float* bias, const float* c_in, float* h_out,
                           float* c_out, void* y, long ldy, float* cs, const int* lens, unsigned* status, int B, int n_in, int n_in_pad, int n, int ndir, hipStream_t s) {
  const int K = n_in_pad + n, nkc = cdiv(K, 32);
  ConcatArgs c = {};
  c.x0 = (const uint16_t*)x; c.ld0 = n_in; c.k0 = 0; c.len0 = n_in;
  c.k1 = c.len1 = 0;
  c.x2 = h_in; c.ld2 = n; c.k2 = n_in_pad; c.len2 = n; c.s2 = (long)B * n;
  c.B = B; c.nkc = nkc;
  c.find_cuts();
  SkinnyArgs a = {};
  a.A = (const char*)A; a.B = (const char*)Wfrag; a.bias = bias; a.M = B; a.N = 4 * n; a.K = K; a.frag = 1;
  a.sAz = (long)cdiv(B, 16) * nkc * 512; a.sBz = (long)cdiv(n, 4) * nkc * 512; a.nz = ndir;
  a.n = n; a.h_in = h_in; a.c_in = c_in; a.h_out = h_out; a.c_out = c_out; a.y = (uint16_t*)y; a.ldy = ldy; a.cs = cs; a.lens = lens; a.status = status;
  const size_t state = (size_t)ndir * B * n * 4;
  bool in_place = false;
  for (const void* o : {(const void*)h_out, (const void*)c_out, (const void*)cs})
    in_place |= bytes_overlap(o, state, h_in, state) || bytes_overlap(o, state, x, (size_t)B * n_in * 2);
  in_place |= bytes_overlap(y, (size_t)B * ldy * 2, h_in, state) || bytes_overlap(y, (size_t)B * ldy * 2, x, (size_t)B * n_in * 2);
  if (B <= 16 && nkc <= 16 * kGatherU && !in_place) {
    hipLaunchKernelGGL((few_gather_kernel<kGatherU, true, true>), dim3(cdiv(n, 4), 1, ndir), dim3(1024), 0, s, a, c, 16);
    return hipGetLastError();
  }
  const long total = (long)cdiv(B, 16) * 16 * nkc * 4;
  hipLaunchKernelGGL(concat_frag_kernel<true>, dim3(cdiv(total, 256), ndir), dim3(256), 0, s, c, (uint4*)A, total);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_rows<true, true>(a, 16, cdiv(n, 4), s);
}

hipError_t launch_few_readout(const void* x0, long ld0, int k0, const void* x1, long ld1, int k1, const void* x2, long ld2, int k2, void* A,
                              const void* Wfrag, const float* bias, void* out, long ldo, int B, int R, hipStream_t s) {
  ConcatArgs c = {};
  c.x0 = (const uint16_t*)x0; c.ld0 = ld0; c.k0 = 0; c.len0 = k0;
  c.x1 = (const uint16_t*)x1; c.ld1 = ld1; c.k1 = k0; c.len1 = k1;
  c.x2 = x2; c.ld2 = ld2; c.k2 = k0 + k1; c.len2 = k2;
  const int K = k0 + k1 + k2;
  c.B = B; c.nkc = cdiv(K, 32);
  c.find_cuts();
  SkinnyArgs a = {};
  a.A = (const char*)A; a.B = (const char*)Wfrag; a.C = out; a.bias = bias; a.M = B; a.N = R; a.K = c.nkc * 32; a.ldc = ldo; a.nz = 1;
  a.out_bf16 = 1; a.relu = 1; a.frag = 1;
  const bool in_place = rows_overlap(out, 2 * ldo, 2L * R, x0, 2 * ld0, 2L * k0, B) || rows_overlap(out, 2 * ldo, 2L * R, x1, 2 * ld1, 2L * k1, B) ||
                        rows_overlap(out, 2 * ldo, 2L * R, x2, 2 * ld2, 2L * k2, B);
  if (B <= 16 && c.nkc <= 16 * kGatherU && !in_place) {
    const int ct = few_columns(B, R);
    hipLaunchKernelGGL((few_gather_kernel<kGatherU, false, false>), dim3(cdiv(R, ct)), dim3(1024), 0, s, a, c, ct);
    return hipGetLastError();
  }
  const long total = (long)cdiv(B, 16) * 16 * c.nkc * 4;
  hipLaunchKernelGGL(concat_frag_kernel<false>, dim3(cdiv(total, 256)), dim3(256), 0, s, c, (uint4*)A, total);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_few(a, s);
}

}  // namespace lstm
