// Recurrent loops of narrow layers: all of W_h on one compute unit.
//
// The single-launch kernels of persistent.hip split a layer's units over many compute units and exchange h (or partial sums of Dh)
// through memory in every step, which costs a step of 1 us (bfloat16) or 6 us (float storage) however narrow the layer is: 20 steps
// of the configuration with 64 units took 125 us.  W_h of n <= 128 units fits the registers of ONE compute unit,
// and batch rows do not interact; so here a work-group is all units of FOUR rows, a step's exchange is a pass through LDS and one
// barrier, and nothing has to be resident together - an ordinary launch whatever else runs on the device.
//
// The product with four rows is what the 4 x 4 x k MFMA with 16 blocks is for: A = four rows of one block, broadcast to all blocks
// (cbsz = 4, abid = the block), B = a column per lane, so an instruction multiplies 4 rows x 64 columns and no row is padding.
// Wavefront w owns units 16 w .. 16 w + 15.  Forward its 64 columns are the four gates of those units (lane = 16 gate + unit) and k
// runs over all units; backward its k are the four gates of its own units - the dz it has just computed - and it covers all n
// outputs, whose shares the wavefronts add through LDS.  A lane's W_h registers: n floats (n / 2 for bfloat16), read once from
// memory as it lies there: no packing pass, no ring, no initial state kernel.
//
// What bounds a step is its chain: LDS read, n MFMAs of 8 clocks (n / 4 bfloat16), gate non-linearities, LDS write, barrier.  Inputs of a
// frame are asked for kAhead frames earlier (a step is shorter than a load from memory).  Four rows of n = 64, float: 0.59 us a step forward, 0.78 backward, and
// 6.5 and 7.5 us to start (W_h, the first inputs); four chains of MFMAs instead of two made no step shorter.
#include "recurrent_dev.h"
#include <type_traits>

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
constexpr int kRows = 4;                 // rows per work-group: what an MFMA of 4 x 4 blocks holds
constexpr int kAhead = 4;                // frames between asking for a frame's inputs and using them

// f(integral_constant<0>) ... f(integral_constant<N - 1>): a loop whose counter is a constant expression in the body
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}
template <int BLOCK>
__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, BLOCK, 0); }
template <int BLOCK>
__device__ __forceinline__ f32x4 mma4(u32x2 a, u32x2 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 4, BLOCK, 0);
}
// Transposes 4 registers x 4 groups of 16 lanes: register v of lane group g -> register g of lane group v.
__device__ __forceinline__ void transpose_groups(f32x4& x) {
  const u32x2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[0]), __float_as_uint(x[2]), false, false);
  const u32x2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[1]), __float_as_uint(x[3]), false, false);
  const u32x2 c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const u32x2 d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  x = (f32x4){__uint_as_float(c[0]), __uint_as_float(c[1]), __uint_as_float(d[0]), __uint_as_float(d[1])};
}

// Between the loads and what looks at them: without it the compiler puts each load into a branch of its own (a column or k past the end needs none) and
// waits for it there, 64 trips to memory one after the other (n = 64, float, 20 steps: forward 23.5 us, 18.5 with them all in flight).
template <typename V> __device__ __forceinline__ void all_in_flight(V& v) { asm volatile("" : "+v"(v)); }

template <typename T> struct Elem;       // an MFMA operand register and what a lane loads for it
template <> struct Elem<float> {
  typedef float reg;                     // one k
  static constexpr int kPer = 1;
};
template <> struct Elem<bf16_t> {
  typedef u32x2 reg;                     // four k
  static constexpr int kPer = 4;
};
__device__ __forceinline__ u32x2 pack4(uint16_t a, uint16_t b, uint16_t c, uint16_t d) { return (u32x2){a | ((unsigned)b << 16), c | ((unsigned)d << 16)}; }

// NW wavefronts: n <= 16 NW, NW a multiple of 4
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void small_fwd_kernel(SmallFwdArgs a) {
  typedef typename Elem<T>::reg reg;
  constexpr int K = 16 * NW, kPer = Elem<T>::kPer, NR = K / kPer;       // B registers per lane: register 16 j + b is block b of group j
  // h of the four rows, as the A operand wants it: [k group][lane = 4 block + row] x (16 bytes float: blocks of four groups; 8 bytes
  // bfloat16: four k of one group)
  __shared__ __attribute__((aligned(16))) char hbuf[2][K * kRows * sizeof(T)];
  const SmallFwdDir d = a.d[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n, B = a.B, Tn = a.T;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.sync = 0u;      // nothing here waits for another work-group
  const int r = lane >> 4, u = wave * 16 + (lane & 15), b = blockIdx.x * kRows + r;      // pointwise: row r, unit u
  const bool active = b < B && u < n;

  reg w[NR];
  {
    const T* W = (const T*)d.W;
    const int q = lane >> 4;                                   // as a column: gate q of unit u
    const bool col = u < n;
    const long c = col ? (long)q * n + u : 0;
    if constexpr (kPer == 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) w[k] = W[(long)min(k, n - 1) * 4 * n + c];
#pragma unroll
      for (int k = 0; k < K; ++k) { all_in_flight(w[k]); w[k] = col && k < n ? w[k] : 0.f; }
    } else {
      const uint16_t* Wu = (const uint16_t*)W;
      unsigned v[K];
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = Wu[(long)min(k, n - 1) * 4 * n + c];
#pragma unroll
      for (int k = 0; k < K; ++k) { all_in_flight(v[k]); v[k] = col && k < n ? v[k] : 0u; }
#pragma unroll
      for (int i = 0; i < NR; ++i) w[i] = (u32x2){v[4 * i] | (v[4 * i + 1] << 16), v[4 * i + 2] | (v[4 * i + 3] << 16)};       // register 16 j + b: k = 64 j + 4 b .. + 3
    }
  }
  float c = 0.f, h = 0.f;
  int L = 0;
  if (active) {
    if (d.c0) c = d.c0[(long)b * n + u];
    if (d.h0) h = d.h0[(long)b * n + u];
    L = clamp_len(a.lens, b, Tn);
  }
  // where this lane's h goes
  int hpos;
  if constexpr (kPer == 1) hpos = ((((u >> 4) >> 2) * 64 + 4 * (u & 15) + r) * 4 + ((u >> 4) & 3)) * 4;
  else hpos = (((u >> 6) * 64 + 4 * ((u >> 2) & 15) + r) * 4 + (u & 3)) * 2;
  uint16_t h_bits = f2bf_bits(h);
  auto put_h = [&](int buf) __attribute__((always_inline)) {
    if constexpr (kPer == 1) *(float*)(hbuf[buf] + hpos) = h;
    else *(uint16_t*)(hbuf[buf] + hpos) = h_bits;
  };
  put_h(0);
  __syncthreads();

  const long g_step = (long)B * 4 * n, s_step = (long)B * n, bb = active ? b : 0, uu = active ? u : 0;
  float zx[kAhead][4];
  auto fetch = [&](int tau, float (&z)[4]) __attribute__((always_inline)) {     // (past the end: the last frame again)
    const int tc = min(tau, Tn - 1), t = d.rev ? Tn - 1 - tc : tc;
    const float* g = d.gates + t * g_step + bb * 4 * n + uu;
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = __builtin_nontemporal_load(g + q * n);
  };
#pragma unroll
  for (int s = 0; s < kAhead; ++s) fetch(s, zx[s]);

  for (int tau0 = 0; tau0 < Tn; tau0 += kAhead) {
    static_for<kAhead>([&](auto S) __attribute__((always_inline)) {
      constexpr int s = decltype(S)::value;
      const int tau = tau0 + s;
      if (tau >= Tn) return;                                   // (the same for every lane)
      const int t = d.rev ? Tn - 1 - tau : tau;
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
      static_for<NW / 4>([&](auto J) __attribute__((always_inline)) {
        constexpr int j4 = decltype(J)::value;
        if constexpr (kPer == 1) {
          const float4 av = *(const float4*)(hbuf[s & 1] + (j4 * 64 + lane) * 16);
          static_for<16>([&](auto Bk) __attribute__((always_inline)) {
            constexpr int bk = decltype(Bk)::value;
            acc0 = mma4<bk>(av.x, w[(4 * j4 + 0) * 16 + bk], acc0);
            acc1 = mma4<bk>(av.y, w[(4 * j4 + 1) * 16 + bk], acc1);
            acc0 = mma4<bk>(av.z, w[(4 * j4 + 2) * 16 + bk], acc0);
            acc1 = mma4<bk>(av.w, w[(4 * j4 + 3) * 16 + bk], acc1);
          });
        } else {
          const u32x2 av = *(const u32x2*)(hbuf[s & 1] + (j4 * 64 + lane) * 8);
          static_for<8>([&](auto Bk) __attribute__((always_inline)) {
            constexpr int bk = 2 * decltype(Bk)::value;
            acc0 = mma4<bk>(av, w[j4 * 16 + bk], acc0);
            acc1 = mma4<bk + 1>(av, w[j4 * 16 + bk + 1], acc1);
          });
        }
      });
      f32x4 z = acc0 + acc1;
      transpose_groups(z);                                     // lane (row r, unit u): its four gates
      const bool valid = t < L;                                // (L is 0 in lanes without a cell)
      const float zh[4] = {z[0], z[1], z[2], z[3]};
      const CellOut o = lstm_cell(zh, zx[s], c);
      const float h_before = h;
      const uint16_t h_before_bits = h_bits;
      if (valid) { c = o.c; h = o.h; h_bits = f2bf_bits(h); }
      put_h((s & 1) ^ 1);
      if (active) {
        const long fr = (long)t * s_step + (long)b * n + u;
        if constexpr (kPer == 1) {
          ((float*)d.y)[((long)t * B + b) * d.ldy + u] = valid ? h : 0.f;
          if (d.hprev) ((float*)d.hprev)[((long)t * B + b) * d.ldh + u] = h_before;
        } else {
          ((uint16_t*)d.y)[((long)t * B + b) * d.ldy + u] = valid ? h_bits : (uint16_t)0;
          if (d.hprev) ((uint16_t*)d.hprev)[((long)t * B + b) * d.ldh + u] = h_before_bits;
        }
        if (d.cs) __builtin_nontemporal_store(c, d.cs + fr);
        if (valid && a.write_gates) {
          float* g = d.gates + t * g_step + (long)b * 4 * n + u;
          __builtin_nontemporal_store(o.gi, g);
          __builtin_nontemporal_store(o.gf, g + n);
          __builtin_nontemporal_store(o.gg, g + 2 * n);
          __builtin_nontemporal_store(o.go, g + 3 * n);
        }
      }
      fetch(tau + kAhead, zx[s]);
      __syncthreads();
    });
  }
  if (active) {
    if (d.hT) d.hT[(long)b * n + u] = h;
    if (d.cT) d.cT[(long)b * n + u] = c;
  }
}

template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void small_bwd_kernel(SmallBwdArgs a) {
  typedef typename Elem<T>::reg reg;
  constexpr int K = 16 * NW, CG = NW / 4, kPer = Elem<T>::kPer;         // CG: groups of 64 outputs
  __shared__ __attribute__((aligned(16))) float red[2][NW][CG][64][kRows];        // [wavefront][output][row]: shares of Dh
  __shared__ __attribute__((aligned(16))) char turn[NW][64 * 16];                 // dz of a wavefront's units, turned into the A operand
  const SmallBwdDir d = a.d[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n, B = a.B, Tn = a.T;
  const int r = lane >> 4, u = wave * 16 + (lane & 15), b = blockIdx.x * kRows + r;
  const bool active = b < B && u < n;

  // register (cg, q, bk) (float) / (cg, bk) (bfloat16, the four gates in it): output cg * 64 + lane, unit wave * 16 + bk
  reg w[CG * (kPer == 1 ? 64 : 16)];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) {
    const int out = cg * 64 + lane;
    const T* W = (const T*)d.W + (long)min(out, n - 1) * 4 * n;
    // (W_h is 16-byte aligned, and so is the second direction of it.  A lane reads a row of its own: loads of 16 bytes where rows allow it, a quarter of the cache lines to look up; n = 64, float: 4.8 us of 27.5, n = 128 20 of 65)
    if constexpr (kPer == 1) {
      if (n % 4 == 0) {
        f32x4 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = *(const f32x4*)(W + (i >> 2) * n + min(wave * 16 + 4 * (i & 3), n - 4));
#pragma unroll
        for (int i = 0; i < 64; ++i) {
          if (i % 4 == 0) all_in_flight(v[i >> 2]);
          w[cg * 64 + i] = v[i >> 2][i & 3];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 64; ++i) w[cg * 64 + i] = W[(i >> 4) * n + min(wave * 16 + (i & 15), n - 1)];
      }
#pragma unroll
      for (int i = 0; i < 64; ++i) { all_in_flight(w[cg * 64 + i]); w[cg * 64 + i] = out < n && wave * 16 + (i & 15) < n ? w[cg * 64 + i] : 0.f; }
    } else {
      unsigned v[64];
      if (n % 8 == 0) {
        typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
        u32x4 x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = *(const u32x4*)((const uint16_t*)W + (i >> 1) * n + min(wave * 16 + 8 * (i & 1), n - 8));
#pragma unroll
        for (int i = 0; i < 64; ++i) {
          if (i % 8 == 0) all_in_flight(x[i >> 3]);
          v[i] = (i & 1) ? x[i >> 3][(i >> 1) & 3] >> 16 : x[i >> 3][(i >> 1) & 3] & 0xffffu;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 64; ++i) v[i] = ((const uint16_t*)W)[(i >> 4) * n + min(wave * 16 + (i & 15), n - 1)];
      }
#pragma unroll
      for (int i = 0; i < 64; ++i) { all_in_flight(v[i]); v[i] = out < n && wave * 16 + (i & 15) < n ? v[i] : 0u; }
#pragma unroll
      for (int bk = 0; bk < 16; ++bk) w[cg * 16 + bk] = (u32x2){v[bk] | (v[16 + bk] << 16), v[32 + bk] | (v[48 + bk] << 16)};
    }
  }
  // the error word (nothing here waits for another work-group) and the counters of the products behind this loop (gemm_tiny.hip)
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.sync = 0u;
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = tid; i < a.ncounters; i += 64 * NW) a.counters[i] = 0u;
  float Dh = 0.f, Dc = 0.f, dbsum[4] = {0.f, 0.f, 0.f, 0.f};
  int L = 0;
  if (active) {
    if (d.dhT) Dh = d.dhT[(long)b * n + u];
    if (d.dcT) Dc = d.dcT[(long)b * n + u];
    L = clamp_len(a.lens, b, Tn);
  }
  const long g_step = (long)B * 4 * n, s_step = (long)B * n, bb = active ? b : 0, uu = active ? u : 0;
  struct In { float gi, gf, gg, go, c_prev, dy; uint16_t dy_bits; };            // c_prev: cell state entering the frame
  auto frame = [&](int tau) { return d.rev ? Tn - 1 - tau : tau; };
  // Cell state after step tau (before the first: the initial one; if there is none, anything: `entering` knows).  One load whichever it is: of a load
  // in a branch the compiler waits for the value where the paths meet, a trip to memory in every step (n = 64, float: 1.00 -> 0.78 us a step, bfloat16 0.74 -> 0.66).
  const float* const before = d.c0 ? d.c0 : d.cs;
  const long lane_s = bb * n + uu, lane_y = bb * d.lddy + uu, y_step = (long)B * d.lddy;
  auto state = [&](int tau) __attribute__((always_inline)) {
    return __builtin_nontemporal_load((tau >= 0 ? d.cs + (long)frame(tau) * s_step : before) + lane_s);
  };
  auto entering = [&](int tau, float c_prev) __attribute__((always_inline)) { return tau > 0 || d.c0 ? c_prev : 0.f; };
  auto fetch = [&](int tau, In& in) __attribute__((always_inline)) {            // (before the beginning: the first frame again)
    const int tc = max(tau, 0), t = frame(tc);
    const float* g = d.gates + t * g_step + bb * 4 * n + uu;
    in.gi = __builtin_nontemporal_load(g); in.gf = __builtin_nontemporal_load(g + n);
    in.gg = __builtin_nontemporal_load(g + 2 * n); in.go = __builtin_nontemporal_load(g + 3 * n);
    in.c_prev = state(tc - 1);
    if constexpr (kPer == 1) in.dy = ((const float*)d.dy)[t * y_step + lane_y];
    else in.dy_bits = ((const uint16_t*)d.dy)[t * y_step + lane_y];
  };
  In in[kAhead];
#pragma unroll
  for (int s = 0; s < kAhead; ++s) fetch(Tn - 1 - s, in[s]);
  float c_new = state(Tn - 1);

  // Dh of the rows that had a frame in the last step, from that step's dz (already in `turn`)
  auto collect = [&](int buf, bool take) __attribute__((always_inline)) {
    f32x4 acc[CG][2];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) acc[cg][0] = acc[cg][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if constexpr (kPer == 1) {
      const float4 av = *(const float4*)(turn[wave] + lane * 16);
      static_for<16>([&](auto Bk) __attribute__((always_inline)) {
        constexpr int bk = decltype(Bk)::value;
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          acc[cg][0] = mma4<bk>(av.x, w[(cg * 4 + 0) * 16 + bk], acc[cg][0]);
          acc[cg][1] = mma4<bk>(av.y, w[(cg * 4 + 1) * 16 + bk], acc[cg][1]);
          acc[cg][0] = mma4<bk>(av.z, w[(cg * 4 + 2) * 16 + bk], acc[cg][0]);
          acc[cg][1] = mma4<bk>(av.w, w[(cg * 4 + 3) * 16 + bk], acc[cg][1]);
        }
      });
    } else {
      const u32x2 av = *(const u32x2*)(turn[wave] + lane * 8);
      static_for<8>([&](auto Bk) __attribute__((always_inline)) {
        constexpr int bk = 2 * decltype(Bk)::value;
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          acc[cg][0] = mma4<bk>(av, w[cg * 16 + bk], acc[cg][0]);
          acc[cg][1] = mma4<bk + 1>(av, w[cg * 16 + bk + 1], acc[cg][1]);
        }
      });
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) *(f32x4*)&red[buf][wave][cg][lane][0] = acc[cg][0] + acc[cg][1];
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) s += red[buf][v][u >> 6][u & 63][r];
    if (take) Dh = s;
  };

  for (int tau0 = Tn - 1; tau0 >= 0; tau0 -= kAhead) {
    static_for<kAhead>([&](auto S) __attribute__((always_inline)) {
      constexpr int s = decltype(S)::value;
      const int tau = tau0 - s;
      if (tau < 0) return;                                     // (the same for every lane)
      const int t = frame(tau);
      if (tau < Tn - 1) collect(s & 1, frame(tau + 1) < L);
      const bool valid = t < L;
      float dz[4] = {0.f, 0.f, 0.f, 0.f};
      const float c_prev = entering(tau, in[s].c_prev), dy = kPer == 1 ? in[s].dy : bf_bits2f(in[s].dy_bits);
      if (valid) lstm_cell_grad(in[s].gi, in[s].gf, in[s].gg, in[s].go, c_new, c_prev, dy + Dh, Dc, dz);
      c_new = c_prev;
      uint16_t bits[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { dbsum[q] += dz[q]; bits[q] = f2bf_bits(dz[q]); }
      // (LDS operations of a wavefront happen in order: no barrier between this and the read in `collect`)
      if constexpr (kPer == 1) *(float4*)(turn[wave] + (4 * (lane & 15) + r) * 16) = make_float4(dz[0], dz[1], dz[2], dz[3]);
      else *(u32x2*)(turn[wave] + (4 * (lane & 15) + r) * 8) = pack4(bits[0], bits[1], bits[2], bits[3]);
      asm volatile("" ::: "memory");
      if (active) {
        const long o = t * g_step + (long)b * 4 * n + u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (kPer == 1) ((float*)d.DZ)[o + q * n] = dz[q];
          else ((uint16_t*)d.DZ)[o + q * n] = bits[q];
        }
      }
      fetch(tau - kAhead, in[s]);
    });
  }
  collect(Tn & 1, frame(0) < L);
  if (active) {
    if (d.dh0) d.dh0[(long)b * n + u] = Dh;
    if (d.dc0) d.dc0[(long)b * n + u] = Dc;
  }
  // bias gradient: the four rows of this work-group; into its slice, or, if it is the only one, straight to its place
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float s = dbsum[q];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (r == 0 && u < n && d.db) {
      float* p = gridDim.x == 1 ? d.db + q * n + u : d.dbpart + (long)blockIdx.x * 4 * n + q * n + u;
      *p = gridDim.x == 1 && a.accumulate ? *p + s : s;
    }
  }
}

// wavefronts (a multiple of 4) for n units, or 0 if the layer is too wide for these kernels
int waves_for(int n) { return n <= 64 ? 4 : n <= 128 ? 8 : 0; }

}  // namespace

bool loop_small_ok(int n) { return waves_for(n) != 0; }

hipError_t launch_small_fwd(const SmallFwdArgs& a, bool bf16, hipStream_t s) {
  const dim3 grid(cdiv(a.B, kRows), a.ndir), block(64 * waves_for(a.n));
  const auto kernel = bf16 ? (a.n <= 64 ? small_fwd_kernel<bf16_t, 4> : small_fwd_kernel<bf16_t, 8>)
                           : (a.n <= 64 ? small_fwd_kernel<float, 4> : small_fwd_kernel<float, 8>);
  hipLaunchKernelGGL(kernel, grid, block, 0, s, a);
  return hipGetLastError();
}
hipError_t launch_small_bwd(const SmallBwdArgs& a, bool bf16, hipStream_t s) {
  const dim3 grid(cdiv(a.B, kRows), a.ndir), block(64 * waves_for(a.n));
  const auto kernel = bf16 ? (a.n <= 64 ? small_bwd_kernel<bf16_t, 4> : small_bwd_kernel<bf16_t, 8>)
                           : (a.n <= 64 ? small_bwd_kernel<float, 4> : small_bwd_kernel<float, 8>);
  hipLaunchKernelGGL(kernel, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace lstm
