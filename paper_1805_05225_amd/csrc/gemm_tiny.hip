// The products of narrow layers and short batches, several in one launch.
//
// At 64 units and 80 frames the four products of a layer are 1.3 MFLOP each; a kernel with 128 x 128 tiles in LDS spends 12 - 22 us on
// one of them (a whole tile's MFMAs for a corner of it, one load latency per stage of K) and every launch costs about 5 us
// beside that.  Here a work-group owns 32 x 32 of C, its four wavefronts share K, and operands go from memory straight into MFMA
// fragments, a batch of loads in flight at a time: nothing is staged, so any alignment and leading dimension will do.  Long K over few
// tiles (the weight gradients) is cut into ranges: every range stores its part and counts itself off, the last one to
// arrive adds them in order - no second launch, and the same result whoever is last.  dX, dW_x and dW_h of a layer are one launch.
// With loop_small.hip a training step of a narrow layer (n_in 32, n 64, 20 steps, 4 rows, float) went from 383 to 59 us.
// What bounds it is latency (a launch, one or two rounds of loads); per flop it loads 8 times what the tiled kernels do, which is why
// it ends at kTinyZxMacs and kTinyBwdMacs.
#include "recurrent_dev.h"
#include <algorithm>

namespace lstm {
namespace {

constexpr int kWaves = 4, kT = 32;
typedef float4 __attribute__((aligned(4))) float4_u;
typedef uint4 __attribute__((aligned(2))) uint4_u;

template <typename T> struct Op;
// float: v_mfma 32x32x2, lane = row + 32 half; four instructions take k = 8 kk + 4 half + e
template <> struct Op<float> {
  static constexpr int kK = 8, kPer = 4;                       // k per chunk, per lane
  struct Frag { float v[4]; };
  __device__ static void mma(const Frag& a, const Frag& b, f32x16& c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e], b.v[e], c, 0, 0, 0);
  }
  __device__ static Frag whole(const void* p) { const float4 x = *(const float4_u*)p; return {{x.x, x.y, x.z, x.w}}; }
  __device__ static void set(Frag& f, int e, const void* p, bool ok) { const float x = *(const float*)p; f.v[e] = ok ? x : 0.f; }
  __device__ static void clear(Frag& f) { f = {{0.f, 0.f, 0.f, 0.f}}; }
};
// bfloat16: v_mfma 32x32x16, k = 16 kk + 8 half + e
template <> struct Op<bf16_t> {
  static constexpr int kK = 16, kPer = 8;
  struct Frag { uint16_t v[8]; };
  __device__ static uint4 pack(const Frag& f) {
    return make_uint4(f.v[0] | ((unsigned)f.v[1] << 16), f.v[2] | ((unsigned)f.v[3] << 16), f.v[4] | ((unsigned)f.v[5] << 16), f.v[6] | ((unsigned)f.v[7] << 16));
  }
  __device__ static void mma(const Frag& a, const Frag& b, f32x16& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pack(a)), __builtin_bit_cast(bf16x8, pack(b)), c, 0, 0, 0);
  }
  __device__ static Frag whole(const void* p) {
    const uint4 x = *(const uint4_u*)p;
    return {{(uint16_t)x.x, (uint16_t)(x.x >> 16), (uint16_t)x.y, (uint16_t)(x.y >> 16), (uint16_t)x.z, (uint16_t)(x.z >> 16), (uint16_t)x.w, (uint16_t)(x.w >> 16)}};
  }
  __device__ static void set(Frag& f, int e, const void* p, bool ok) { const uint16_t x = *(const uint16_t*)p; f.v[e] = ok ? x : (uint16_t)0; }
  __device__ static void clear(Frag& f) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f.v[e] = 0;
  }
};

// A lane's share of a chunk: `line` = its row (k-contiguous) or column (k-major) of the operand, inside it by construction; k .. k + kPer - 1.
template <typename T, bool KC>
__device__ __forceinline__ typename Op<T>::Frag load(const char* base, long ld, long line, int k, int K, const int* lens, int Bt, int Tn) {
  constexpr int E = sizeof(T), P = Op<T>::kPer;
  typename Op<T>::Frag f;
  if constexpr (KC) {
    const char* p = base + (line * ld + k) * E;
    if (k + P <= K) return Op<T>::whole(p);
    Op<T>::clear(f);
#pragma unroll
    for (int e = 0; e < P; ++e)
      if (k + e < K) Op<T>::set(f, e, p + e * E, true);
  } else {
#pragma unroll
    for (int e = 0; e < P; ++e) {
      const int kc = min(k + e, K - 1);
      bool ok = k + e < K;
      if (lens) {                                              // (uniform)
        const int t = kc / Bt;
        ok = ok && t < clamp_len(lens, kc - t * Bt, Tn);
      }
      Op<T>::set(f, e, base + ((long)kc * ld + line) * E, ok);
    }
  }
  return f;
}

template <typename T, bool AK, bool BK>
__device__ __forceinline__ void product(const TinyProduct& p, int tile, float (&red)[kWaves][kT][kT + 1], unsigned* counters, float* parts, int first_part) {
  constexpr int E = sizeof(T), U = 4;                          // chunks of a wavefront in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l = lane & 31;
  const int tiles_m = (p.M + kT - 1) / kT, tiles_n = (p.N + kT - 1) / kT;
  const int range = tile % p.ksplit;
  int rest = tile / p.ksplit;
  const int out_tile = rest;                                   // z, tile row, tile column
  const int tn = rest % tiles_n; rest /= tiles_n;
  const int tm = rest % tiles_m, z = rest / tiles_m;
  const int m0 = tm * kT, n0 = tn * kT;
  const int per_seg = (p.K + Op<T>::kK - 1) / Op<T>::kK, chunks = per_seg * p.nseg;
  const int c0 = (int)((long)chunks * range / p.ksplit), c1 = (int)((long)chunks * (range + 1) / p.ksplit);
  const long arow = min(m0 + l, p.M - 1), brow = min(n0 + l, p.N - 1);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int c = c0 + wave; c < c1; c += kWaves * U) {
    typename Op<T>::Frag fa[U], fb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = min(c + u * kWaves, c1 - 1), seg = cc / per_seg, k = (cc - seg * per_seg) * Op<T>::kK + half * Op<T>::kPer;
      fa[u] = load<T, AK>((const char*)p.A + (p.sAz * z + p.sAseg * seg) * E, p.lda, arow, k, p.K, AK ? nullptr : p.lens, p.Bt, p.T);
      fb[u] = load<T, BK>((const char*)p.B + (p.sBz * z + p.sBseg * seg) * E, p.ldb, brow, k, p.K, nullptr, 1, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u * kWaves < c1) Op<T>::mma(fa[u], fb[u], acc);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][8 * (v >> 2) + 4 * half + (v & 3)][l] = acc[v];
  __syncthreads();
  float sum[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = tid + 256 * i, r = idx >> 5, cc = idx & 31;
    sum[i] = (red[0][r][cc] + red[1][r][cc]) + (red[2][r][cc] + red[3][r][cc]);
  }
  if (p.ksplit > 1) {
    __shared__ int last;
    float* mine = parts + (long)(first_part + tile) * (kT * kT);
#pragma unroll
    for (int i = 0; i < 4; ++i) __hip_atomic_store(&mine[tid + 256 * i], sum[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // What a release at device scope does on this device is (1) write the XCD's dirty L2 lines back, (2) wait until every store before it
    // has been acknowledged (vmcnt 0), (3) let the atomic behind it go.  The parts need no (1): a device-scope atomic store is
    // written through (sc1), and it is acknowledged where all XCDs meet, not by the L2 on the way - (2) would order nothing otherwise.
    // Their readers are device-scope atomic loads, which take nothing from an L2 that another XCD may have overtaken, and go out
    // only after the counter's value has come back and the barrier behind it.  So (2) is all there is to do; a whole release costs 80
    // instead of 27 us for the launch.  (vmcnt 0 counts everything: nothing here hangs on the order in which loads and stores
    // are acknowledged, which the single-launch loops have found not to be that of issue.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) last = (int)__hip_atomic_fetch_add(&counters[first_part + out_tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == p.ksplit - 1;
    __syncthreads();
    if (!last) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[i] = 0.f;
    for (int q = 0; q < p.ksplit; ++q) {
      const float* part = parts + (long)(first_part + out_tile * p.ksplit + q) * (kT * kT);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] += __hip_atomic_load(&part[tid + 256 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = tid + 256 * i, m = m0 + (idx >> 5), n = n0 + (idx & 31);
    if (m >= p.M || n >= p.N) continue;
    float v = sum[i] + (p.bias ? p.bias[p.sbiasz * z + n] : 0.f);
    const long o = p.sCz * z + (long)m * p.ldc + n;
    if (p.out_bf16) ((uint16_t*)p.C)[o] = f2bf_bits(v);
    else ((float*)p.C)[o] = p.accumulate ? ((float*)p.C)[o] + v : v;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void gemm_tiny_kernel(TinyGroup g, unsigned* counters, float* parts) {
  __shared__ float red[kWaves][kT][kT + 1];
  int i = 0;
  if (g.count > 1 && (int)blockIdx.x >= g.p[1].tile0) i = 1;
  if (g.count > 2 && (int)blockIdx.x >= g.p[2].tile0) i = 2;
  const TinyProduct& p = g.p[i];
  const int tile = blockIdx.x - p.tile0;
  if (p.a_kcontig && p.b_kcontig) product<T, true, true>(p, tile, red, counters, parts, p.tile0);
  else if (p.a_kcontig) product<T, true, false>(p, tile, red, counters, parts, p.tile0);
  else product<T, false, false>(p, tile, red, counters, parts, p.tile0);
}

long tiles_of(const TinyProduct& p) { return (long)cdiv(p.M, kT) * cdiv(p.N, kT) * p.nz; }
// K ranges: about two work-groups per CU and product, at least 128 k each (a batch of loads of the four wavefronts)
int ranges_of(const TinyProduct& p) {
  const long tiles = std::max(tiles_of(p), 1L);
  return (int)std::max(1L, std::min(512 / tiles, (long)p.K * p.nseg / 128));
}
int plan(TinyGroup& g, bool split) {
  long at = 0;
  for (int i = 0; i < g.count; ++i) {
    g.p[i].ksplit = split ? ranges_of(g.p[i]) : 1;
    g.p[i].tile0 = (int)at;
    at += tiles_of(g.p[i]) * g.p[i].ksplit;
  }
  return (int)at;
}

}  // namespace

long tiny_macs(const TinyProduct& p) { return (long)p.M * p.N * p.nz * p.nseg * p.K; }
int tiny_counters(const TinyGroup& g) {
  TinyGroup c = g;
  return plan(c, true);
}
size_t tiny_parts_bytes(const TinyGroup& g) {
  TinyGroup c = g;
  return (size_t)plan(c, true) * kT * kT * 4;
}
// (parts == NULL: K in one piece, no counters)
hipError_t launch_gemm_tiny(const TinyGroup& g, bool in_bf16, unsigned* counters, float* parts, hipStream_t s) {
  TinyGroup c = g;
  const int blocks = plan(c, parts != nullptr);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(in_bf16 ? gemm_tiny_kernel<bf16_t> : gemm_tiny_kernel<float>, dim3(blocks), dim3(256), 0, s, c, counters, parts);
  return hipGetLastError();
}

}  // namespace lstm
