// Device helpers shared by the per-step and the persistent recurrent kernels.
#pragma once
#include "common.h"

namespace lstm {
namespace {

// Four more k for a 32 x 32 block: K of a product of k-contiguous operands that is 4 more than a multiple of 8 (4n for odd n) ends in half a 16-byte chunk,
// whose other half is the next row's.  The kernels walk the whole chunks and begin their accumulators with these products, operands straight
// from memory (lanes 0-31 four k of a row; lanes 32-63, which hold the next four, zeros).
__device__ __forceinline__ f32x16 mma_last4(uint2 a, uint2 b, f32x16 c) {
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}
// dst[r][c] = src[r][c] for c < C, zero for C <= c < 8 ldd8 (rows made whole 16 bytes).  16 bytes a thread, read at any element
// (9456 rows of 1802 elements: 40 us with an element a thread, 12.8).
__device__ __forceinline__ void pad_rows_body(long idx, const uint16_t* src, uint4* dst, long R, int C, int ldd8) {
  struct __attribute__((packed, aligned(2))) Chunk { uint16_t v[8]; };
  if (idx >= R * ldd8) return;
  const long rr = idx / ldd8;
  const int c0 = (int)(idx - rr * ldd8) * 8;
  const uint16_t* p = src + rr * C + c0;
  Chunk o = {};
  if (c0 + 8 <= C) o = *(const Chunk*)p;
  else {
#pragma unroll
    for (int e = 0; e < 8; ++e) if (c0 + e < C) o.v[e] = p[e];
  }
  dst[idx] = __builtin_bit_cast(uint4, o);
}
// Block `block` (256 threads) of those that clear the regions.
__device__ __forceinline__ void fill_zero_body(const ZeroRegions& r, int block, int tid) {
  int k = 0;
#pragma unroll
  for (int j = 1; j < ZeroRegions::kMax; ++j)
    if (j < r.count && block >= r.first_block[j]) k = j;
  uint32_t* p = (uint32_t*)r.ptr[k];
  const size_t nwords = r.words[k], nb = (size_t)(r.first_block[k + 1] - r.first_block[k]);
  for (size_t i = (size_t)(block - r.first_block[k]) * 256 + tid; i < nwords; i += nb * 256) p[i] = 0u;
}
// Frame map of a batch of end-padded sequences (see launch_frame_map), the work of one block of 256 threads: four time steps,
// one wavefront each.  Shared by the kernel of its own and by the set-up kernel of the single-launch loops.
__device__ __forceinline__ void frame_map_body(int block, const int* lens, int T, int B, int* fidx, int* count) {
  const int lane = threadIdx.x & 63;
  const int t = block * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  // kept frames before time t: sum over b of min(len_b, t)
  long before = 0, all = 0;
  for (int b = lane; b < B; b += 64) {
    int L = lens[b];
    L = L < 0 ? 0 : (L > T ? T : L);
    before += L < t ? L : t;
    all += L;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    before += __shfl_xor(before, o);
    all += __shfl_xor(all, o);
  }
  if (t == 0 && lane == 0) {
    count[0] = (int)all;
    count[1] = (int)((all + 63) / 64 * 64);
  }
  int base = (int)before;
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int b = b0 + lane;
    bool keep = false;
    if (b < B) {
      int L = lens[b];
      L = L < 0 ? 0 : (L > T ? T : L);
      keep = t < L;
    }
    const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
    const int mine = base + __popcll(m & ((1ull << lane) - 1ull));
    if (keep) fidx[mine] = t * B + b;
    base += __popcll(m);
  }
}

template <typename T> struct Mma16;
template <> struct Mma16<bf16_t> {
  __device__ static f32x4 run(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma16<float> {
  __device__ static f32x4 run(uint4 a, uint4 b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

// element offset (in elements of T) of (row, k) inside a fragment-ordered buffer with nkc chunks per row tile
template <typename T>
__device__ __forceinline__ long frag_offset(int row, int k, int nkc) {
  constexpr int E = Store<T>::kPerChunk, KC = 4 * E;
  int rt = row >> 4, r = row & 15;
  int kc = k / KC, rem = k - kc * KC;
  int g = rem / E, e = rem - g * E;
  return ((((long)rt * nkc + kc) * 64 + g * 16 + r) * E + e);
}

// Reciprocals through the hardware approximation (1 ulp): a correctly rounded float division is ten dependent
// instructions, and with one wavefront per SIMD the recurrent kernels pay for every one of them in every step.
__device__ __forceinline__ float sigmoidf_(float x) { return __builtin_amdgcn_rcpf(1.f + __expf(-x)); }
__device__ __forceinline__ float tanhf_(float x) { return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + __expf(2.f * x)); }
__device__ __forceinline__ int clamp_len(const int* lens, int b, int T) {
  if (!lens) return T;
  int L = lens[b];
  return L < 0 ? 0 : (L > T ? T : L);
}


// One LSTM cell update in float.  zh = h W_h part, zx = x W_x + b part, both ordered i|f|g|o.
struct CellOut { float gi, gf, gg, go, c, h; };
__device__ __forceinline__ CellOut lstm_cell(const float (&zh)[4], const float (&zx)[4], float c_prev) {
  CellOut o;
  o.gi = sigmoidf_(zh[0] + zx[0]);
  o.gf = sigmoidf_(zh[1] + zx[1]);
  o.gg = tanhf_(zh[2] + zx[2]);
  o.go = sigmoidf_(zh[3] + zx[3]);
  o.c = o.gf * c_prev + o.gi * o.gg;
  o.h = o.go * tanhf_(o.c);
  return o;
}
// Gate gradients of one valid frame.  dh = dy + carried Dh; Dc is updated in place.
__device__ __forceinline__ void lstm_cell_grad(float gi, float gf, float gg, float go, float c_new, float c_prev, float dh,
                                               float& Dc, float (&dz)[4]) {
  const float tc = tanhf_(c_new);
  const float dc = Dc + dh * go * (1.f - tc * tc);
  Dc = dc * gf;
  dz[0] = dc * gg * gi * (1.f - gi);
  dz[1] = dc * c_prev * gf * (1.f - gf);
  dz[2] = dc * gi * (1.f - gg * gg);
  dz[3] = dh * tc * go * (1.f - go);
}

// W_h for the per-step and the float single-launch forward kernels.
// forward: chunk index = ((dir*ntiles + tile)*2 + ct)*nkc + kc)*64 + lane ; column ct*16 + (lane%16) of the
// work-group's 32 columns is gate q = col/8, unit tile*8 + col%8.
template <typename T>
__device__ __forceinline__ void pack_wh_fwd_body(long idx, const T* W, uint4* out, int n, int nkc, long total) {
  constexpr int E = Store<T>::kPerChunk, KC = 4 * E;
  if (idx >= total) return;
  int lane = idx & 63;
  long rest = idx >> 6;
  int kc = rest % nkc; rest /= nkc;
  int ct = rest & 1; rest >>= 1;
  int ntiles = (n + 7) / 8;
  int tile = rest % ntiles;
  int dir = rest / ntiles;
  int col = ct * 16 + (lane & 15), g = lane >> 4;
  int q = col >> 3, unit = tile * 8 + (col & 7);
  const T* Wd = W + (long)dir * n * 4 * n;
  T v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    int k = kc * KC + g * E + e;
    v[e] = (k < n && unit < n) ? Wd[(long)k * 4 * n + q * n + unit] : (T)0.f;
  }
  out[idx] = *(uint4*)v;
}

}  // namespace
}  // namespace lstm
