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
// runs over all units; backward its k are the four gates of its own units - the dz it has just computed, in lane 4 unit + row, which is an A
// operand as it stands - and it covers all n outputs, whose shares the wavefronts add through LDS.  A lane's W_h registers: n floats (n / 2 for
// bfloat16), read once from memory as it lies there: no packing pass, no ring, no initial state kernel.
//
// What bounds a step is its chain: LDS read, n MFMAs of 8 clocks (n / 4 bfloat16), gate non-linearities, LDS write, barrier.  All else is kept
// out of it: a frame's outputs are stored in the next step, behind its products, its inputs are asked for kAhead frames earlier, what the gate
// gradients take from the inputs alone is computed behind the products of the step before, addresses are scalar pointers that move a frame a step.  And
// no step may wait for loads it has just issued (see walk): a wait before the barrier of every step was a third of it backward.
// Two chains of products (four, for shorter chains, cost more in clearing and adding them than they gave:
// forward 0.56 and 0.39 us for n = 64, backward 0.62 and 0.42).
// us a step, forward and backward, before and now: four rows of n = 64, float 0.59 and 0.79, 0.54 and 0.58; bfloat16 0.48 and 0.72, 0.37 and 0.40; n = 128,
// float 1.36 and 1.60, 1.24 and 1.35 (256 MFMAs a matrix core: 1.0); bfloat16 0.70 and 1.05, 0.60 and 0.75.  6 and 9 us to start (W_h, the first inputs; n = 82,
// bfloat16, four layers of 9 steps, forward only: a call of 84 us is 64 since W_h is read by 16 bytes).
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

__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {      // round to nearest even, low half first
  typedef __attribute__((ext_vector_type(2))) float f32x2_;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_;
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2_){lo, hi}, bf16x2_));
}
__device__ __forceinline__ unsigned bf16_bits(float v) { return pack_bf16x2(v, 0.f) & 0xffffu; }
constexpr unsigned kParked = 0x7ff00000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frame_of(const void* base, unsigned bytes) { return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000); }
// a barrier behind this wavefront's LDS operations (not behind its loads and stores)
__device__ __forceinline__ void meet() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);                          // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// step(k, integral_constant<k % kAhead>) for k < steps, in whole rounds and a rest of its own: where a step may be passed over (or the loop left) inside a
// round, the compiler's wait counts allow for paths on which less was issued, and every step waits for the loads it has just asked for.
template <typename F>
__device__ __forceinline__ void walk(int steps, F&& step) {
  int k = 0;
  for (; k + kAhead <= steps; k += kAhead) static_for<kAhead>([&](auto S) __attribute__((always_inline)) { step(k + decltype(S)::value, S); });
  static_for<kAhead - 1>([&](auto S) __attribute__((always_inline)) { if (k + decltype(S)::value < steps) step(k + decltype(S)::value, S); });
}

// NW wavefronts: n <= 16 NW, NW a multiple of 4
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void small_fwd_kernel(SmallFwdArgs a) {
  typedef typename Elem<T>::reg reg;
  constexpr int K = 16 * NW, kPer = Elem<T>::kPer, NR = K / kPer;       // B registers per lane: register 16 j + b is block b of group j
  // h of the four rows, as the A operand wants it: [k group][lane = 4 block + row] x (16 bytes float: blocks of four groups; 8 bytes
  // bfloat16: four k of one group)
  __shared__ __attribute__((aligned(16))) char hbuf[2][K * kRows * sizeof(T)];
  __shared__ __attribute__((aligned(16))) char wbuf[NW][8192];
  const SmallFwdDir d = a.d[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n, B = a.B, Tn = a.T;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.sync = 0u;      // nothing here waits for another work-group
  const int r = lane >> 4, u = wave * 16 + (lane & 15), b = blockIdx.x * kRows + r;      // pointwise: row r, unit u
  const bool active = b < B && u < n;

  // W_h, first of all that the first steps need (asked for together: one after the other they are four trips to memory).  A lane's column is gate
  // lane / 16 of unit u, four bytes of a row or two: loads of those, K a lane, are 7 us of work for the address unit at n = 128.  So a wavefront fetches its columns'
  // parts of a row by 16 bytes a lane and turns them in LDS.  (Rows past n arrive as zeros, units past n are cleared below; an odd n in bfloat16 has rows
  // that are not whole dwords.)
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  constexpr int kRowLanes = 4 * sizeof(T), kRowsPerLoad = 64 / kRowLanes, kLoads = K / kRowsPerLoad, kPart = 8, kPartRows = kPart * kRowsPerLoad;
  const bool wide = kPer == 1 || n % 2 == 0;
  u32x4 raw[kLoads];
  if (wide) {
    const __amdgpu_buffer_rsrc_t rs = frame_of(d.W, (unsigned)(4 * n * n * sizeof(T)));
    const int seg = lane % kRowLanes, unit = wave * 16 + seg % (kRowLanes / 4) * (16 / (int)sizeof(T));
    const unsigned off = (unsigned)(((lane / kRowLanes) * 4 * n + seg / (kRowLanes / 4) * n + unit) * sizeof(T));
#pragma unroll
    for (int i = 0; i < kLoads; ++i) raw[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + (unsigned)(i * kRowsPerLoad * 4 * n * sizeof(T)), 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);

  // Frames go by scalar pointers that move a frame a step, lanes by offsets inside the work-group's rows that never change: a descriptor covers the
  // rows' part of one frame, a lane without a cell is parked outside (reads zeros, stores nothing), an absent array is an empty one.
  const int b0 = blockIdx.x * kRows, rows = min(kRows, B - b0);
  const long dir = d.rev ? -1 : 1, first = d.rev ? Tn - 1 : 0;
  const long g_step = dir * B * 16 * n, y_step = dir * B * d.ldy * (long)sizeof(T), s_step = dir * B * 4 * n, h_step = dir * B * d.ldh * (long)sizeof(T);
  auto at = [&](const void* base, long step, long row_bytes) { return base ? (char*)base + (d.rev ? -step : step) * first + b0 * row_bytes : nullptr; };
  char* g_in = at(d.gates, g_step, 16L * n);                               // frame that is asked for next
  char* g_out = at(d.gates, g_step, 16L * n) - g_step;                     // frame of the step before (stored in the next one)
  char* y_out = at(d.y, y_step, d.ldy * (long)sizeof(T)) - y_step;
  char* c_out = d.cs ? at(d.cs, s_step, 4L * n) - s_step : nullptr;
  char* h_out = d.hprev ? at(d.hprev, h_step, d.ldh * (long)sizeof(T)) - h_step : nullptr;
  const unsigned g_bytes = rows * 16u * n, y_bytes = (unsigned)(rows * d.ldy * sizeof(T)), s_bytes = rows * 4u * n, h_bytes = (unsigned)(rows * d.ldh * sizeof(T));
  const unsigned g_off = active ? (r * 4u * n + u) * 4u : kParked, s_off = active ? (r * n + u) * 4u : kParked;
  const unsigned y_off = active ? (unsigned)((r * d.ldy + u) * sizeof(T)) : kParked, h_off = active ? (unsigned)((r * d.ldh + u) * sizeof(T)) : kParked;
  const unsigned gate = 4u * n;
  const unsigned l_off = active ? 4u * b : kParked;
  const unsigned len_bits = __builtin_amdgcn_raw_buffer_load_b32(frame_of(a.lens, a.lens ? 4u * B : 0u), l_off, 0, 0);
  float c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.c0 ? d.c0 + (long)b0 * n : nullptr, d.c0 ? s_bytes : 0u), s_off, 0, 0));
  float h = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.h0 ? d.h0 + (long)b0 * n : nullptr, d.h0 ? s_bytes : 0u), s_off, 0, 0));
  float zx[kAhead][4];
  int asked = 0;
  auto fetch = [&](float (&z)[4]) __attribute__((always_inline)) {        // (past the end: the last frame again)
    const __amdgpu_buffer_rsrc_t rs = frame_of(g_in, g_bytes);
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, g_off, q * gate, 2));
    ++asked;
    g_in += asked < Tn ? g_step : 0;
  };
#pragma unroll
  for (int s = 0; s < kAhead - 1; ++s) {
    fetch(zx[s]);
    __builtin_amdgcn_sched_barrier(0);                                     // (in this order: the first step's are waited for first)
  }

  reg w[NR];                                                   // bfloat16: register 16 j + b: k = 64 j + 4 b .. + 3
  if (wide) {
#pragma unroll
    for (int p = 0; p < kLoads / kPart; ++p) {                 // (LDS operations of a wavefront happen in order)
#pragma unroll
      for (int i = 0; i < kPart; ++i) *(u32x4*)(wbuf[wave] + i * 1024 + lane * 16) = raw[p * kPart + i];
      if constexpr (kPer == 1) {
#pragma unroll
        for (int k = 0; k < kPartRows; ++k) w[p * kPartRows + k] = *(const float*)(wbuf[wave] + k * 256 + lane * 4);
      } else {
        const char* from = wbuf[wave] + ((lane & 15) >> 2) * 128 + (lane >> 4) * 32 + (lane & 3) * 8;      // (the layout of this read: gemm_nt.hip)
#pragma unroll
        for (int i = 0; i < kPartRows / 4; ++i)
          w[p * (kPartRows / 4) + i] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(from + i * 512)));
      }
      asm volatile("" ::: "memory");
    }
  } else if constexpr (kPer != 1) {
    const uint16_t* W = (const uint16_t*)d.W + (u < n ? (long)(lane >> 4) * n + u : 0);
    unsigned v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = W[(long)min(k, n - 1) * 4 * n];
#pragma unroll
    for (int k = 0; k < K; ++k) { all_in_flight(v[k]); v[k] = k < n ? v[k] : 0u; }
#pragma unroll
    for (int i = 0; i < NR; ++i) w[i] = (u32x2){v[4 * i] | (v[4 * i + 1] << 16), v[4 * i + 2] | (v[4 * i + 3] << 16)};
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    if constexpr (kPer == 1) w[i] = u < n ? w[i] : 0.f;
    else w[i] = u < n ? w[i] : (u32x2){0u, 0u};
  }
  const int L = !active ? 0 : a.lens ? max(0, min((int)len_bits, Tn)) : Tn;
  // where this lane's h goes
  int hpos;
  if constexpr (kPer == 1) hpos = ((((u >> 4) >> 2) * 64 + 4 * (u & 15) + r) * 4 + ((u >> 4) & 3)) * 4;
  else hpos = (((u >> 6) * 64 + 4 * ((u >> 2) & 15) + r) * 4 + (u & 3)) * 2;
  unsigned h_bits = bf16_bits(h);
  auto put_h = [&](int buf) __attribute__((always_inline)) {
    if constexpr (kPer == 1) *(float*)(hbuf[buf] + hpos) = h;
    else *(uint16_t*)(hbuf[buf] + hpos) = (uint16_t)h_bits;
  };
  put_h(0);
  __syncthreads();


  // What a step leaves: stored in the next one, behind its LDS read and its products, where the chain does not wait for it.
  CellOut o = {};
  unsigned before = 0u;
  bool was_valid = false;
  auto store = [&](int k, bool some) __attribute__((always_inline)) {     // output k of 7
    if (k == 0) {
      const __amdgpu_buffer_rsrc_t rs = frame_of(y_out, some ? y_bytes : 0u);
      if constexpr (kPer == 1) __builtin_amdgcn_raw_buffer_store_b32(was_valid ? __float_as_uint(h) : 0u, rs, y_off, 0, 0);
      else __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(was_valid ? h_bits : 0u), rs, y_off, 0, 0);
    } else if (k == 1) {
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c), frame_of(c_out, some && c_out ? s_bytes : 0u), s_off, 0, 2);
    } else if (k == 2) {
      const __amdgpu_buffer_rsrc_t rs = frame_of(h_out, some && h_out ? h_bytes : 0u);
      if constexpr (kPer == 1) __builtin_amdgcn_raw_buffer_store_b32(before, rs, h_off, 0, 0);
      else __builtin_amdgcn_raw_buffer_store_b16((unsigned short)before, rs, h_off, 0, 0);
    } else {
      const float v = k == 3 ? o.gi : k == 4 ? o.gf : k == 5 ? o.gg : o.go;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), frame_of(g_out, some && a.write_gates ? g_bytes : 0u), was_valid ? g_off : kParked, (k - 3) * gate, 2);
    }
    if (k == 6) {
      y_out += y_step; g_out += g_step; c_out += c_out ? s_step : 0; h_out += h_out ? h_step : 0;
    }
  };
  int t = (int)first;
  auto step = [&](int tau, auto S) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
    typedef typename std::conditional<kPer == 1, f32x4, u32x2>::type operand;
    operand av[NW / 4];
#pragma unroll
    for (int j4 = 0; j4 < NW / 4; ++j4) av[j4] = *(const operand*)(hbuf[s & 1] + (j4 * 64 + lane) * sizeof(operand));
    __builtin_amdgcn_sched_barrier(0);
    const bool some = tau > 0;
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    // (the first two outputs while the LDS read is on its way, the others and the next inputs behind products)
    store(0, some);
    store(1, some);
    auto behind = [&](int i) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      if (i < 5) store(i + 2, some);
      if (i == 5) fetch(zx[(s + kAhead - 1) % kAhead]);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<NW / 4>([&](auto J) __attribute__((always_inline)) {
      constexpr int j4 = decltype(J)::value;
      if constexpr (kPer == 1) {
        static_for<16>([&](auto Bk) __attribute__((always_inline)) {
          constexpr int bk = decltype(Bk)::value;
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i & 1] = mma4<bk>(av[j4][i], w[(4 * j4 + i) * 16 + bk], acc[i & 1]);
          if (j4 == 0) behind(bk);
        });
      } else {
        static_for<4>([&](auto Bk) __attribute__((always_inline)) {
          constexpr int bk = 4 * decltype(Bk)::value;
          acc[0] = mma4<bk>(av[j4], w[j4 * 16 + bk], acc[0]);
          acc[1] = mma4<bk + 1>(av[j4], w[j4 * 16 + bk + 1], acc[1]);
          acc[0] = mma4<bk + 2>(av[j4], w[j4 * 16 + bk + 2], acc[0]);
          acc[1] = mma4<bk + 3>(av[j4], w[j4 * 16 + bk + 3], acc[1]);
          if (j4 == 0 && bk < 12) { behind(bk / 2); behind(bk / 2 + 1); }
        });
      }
    });
    f32x4 z = acc[0] + acc[1];
    transpose_groups(z);                                     // lane (row r, unit u): its four gates
    was_valid = t < L;                                       // (L is 0 in lanes without a cell)
    const float zh[4] = {z[0], z[1], z[2], z[3]};
    o = lstm_cell(zh, zx[s], c);
    before = kPer == 1 ? __float_as_uint(h) : h_bits;
    c = was_valid ? o.c : c;
    h = was_valid ? o.h : h;
    h_bits = bf16_bits(h);
    put_h((s & 1) ^ 1);
    t += d.rev ? -1 : 1;
    meet();
  };
  if (Tn > 0) {
    walk(Tn, step);
#pragma unroll
    for (int k = 0; k < 7; ++k) store(k, true);
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
  const SmallBwdDir d = a.d[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = a.n, B = a.B, Tn = a.T;
  // (row and unit of a lane as an A operand has them, lane = 4 block + row: its dz is one as it stands)
  const int r = lane & 3, u = wave * 16 + (lane >> 2), b = blockIdx.x * kRows + r;
  const bool active = b < B && u < n;

  // (scalar pointers and descriptors as forward; processing order is the forward step's, walked backwards)
  const int b0 = blockIdx.x * kRows, rows = min(kRows, B - b0);
  const long dir = d.rev ? 1 : -1, last = d.rev ? 0 : Tn - 1;              // frames of the steps from Tn - 1 down
  const long g_step = dir * B * 16 * n, s_step = dir * B * 4 * n, y_step = dir * B * d.lddy * (long)sizeof(T), z_step = dir * B * 4 * n * (long)sizeof(T);
  auto at = [&](const void* base, long step, long row_bytes) { return (char*)base + (d.rev ? step : -step) * last + b0 * row_bytes; };
  char* g_in = at(d.gates, g_step, 16L * n);
  char* y_in = at(d.dy, y_step, d.lddy * (long)sizeof(T));
  char* c_in = at(d.cs, s_step, 4L * n);                                   // the state that leaves a frame
  char* z_out = at(d.DZ, z_step, 4L * n * (long)sizeof(T));
  const unsigned g_bytes = rows * 16u * n, y_bytes = (unsigned)(rows * d.lddy * sizeof(T)), s_bytes = rows * 4u * n, z_bytes = (unsigned)(rows * 4 * n * sizeof(T));
  const unsigned g_off = active ? (r * 4u * n + u) * 4u : kParked, s_off = active ? (r * n + u) * 4u : kParked;
  const unsigned y_off = active ? (unsigned)((r * d.lddy + u) * sizeof(T)) : kParked, z_off = active ? (unsigned)((r * 4 * n + u) * sizeof(T)) : kParked;
  const unsigned gate = 4u * n, z_gate = (unsigned)(n * sizeof(T));
  const unsigned l_off = active ? 4u * b : kParked;
  const unsigned len_bits = __builtin_amdgcn_raw_buffer_load_b32(frame_of(a.lens, a.lens ? 4u * B : 0u), l_off, 0, 0);
  float Dh = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.dhT ? d.dhT + (long)b0 * n : nullptr, d.dhT ? s_bytes : 0u), s_off, 0, 0));
  float Dc = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.dcT ? d.dcT + (long)b0 * n : nullptr, d.dcT ? s_bytes : 0u), s_off, 0, 0));
  float dbsum[4] = {0.f, 0.f, 0.f, 0.f};
  // c_prev: cell state entering the frame.  (dy as it is loaded: widened, it would be waited for at the loop's end.)
  struct In { float gi, gf, gg, go, c_prev; typename std::conditional<kPer == 1, unsigned, unsigned short>::type dy_bits; };
  auto state = [&]() __attribute__((always_inline)) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(c_in, c_in ? s_bytes : 0u), s_off, 0, 2)); };
  char* const c_first = d.c0 ? (char*)(d.c0 + (long)b0 * n) : nullptr;         // (none: zeros)
  int asked = Tn - 1;                                                          // step whose inputs are asked for next
  float c_new = state();
  auto fetch = [&](In& in) __attribute__((always_inline)) {                    // (before the beginning: the first frame again)
    const __amdgpu_buffer_rsrc_t rg = frame_of(g_in, g_bytes), ry = frame_of(y_in, y_bytes);
    in.gi = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, g_off, 0, 2));
    in.gf = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, g_off, gate, 2));
    in.gg = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, g_off, 2 * gate, 2));
    in.go = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, g_off, 3 * gate, 2));
    c_in = asked > 0 ? c_in + s_step : c_first;                                // the state that enters: the one that leaves the frame before, or the initial one
    in.c_prev = state();
    if constexpr (kPer == 1) in.dy_bits = __builtin_amdgcn_raw_buffer_load_b32(ry, y_off, 0, 0);
    else in.dy_bits = __builtin_amdgcn_raw_buffer_load_b16(ry, y_off, 0, 0);
    g_in += asked > 0 ? g_step : 0;
    y_in += asked > 0 ? y_step : 0;
    asked -= asked > 0 ? 1 : 0;
  };
  In in[kAhead];
#pragma unroll
  for (int s = 0; s < kAhead; ++s) {
    fetch(in[s]);
    __builtin_amdgcn_sched_barrier(0);                                         // (in this order: the first step's are waited for first)
  }

  // register (cg, q, bk) (float) / (cg, bk) (bfloat16, the four gates in it): output cg * 64 + lane, unit wave * 16 + bk
  // A lane reads a row of its own, 16 bytes at a time: a quarter of the cache lines to look up, an eighth of the loads of single bfloat16 (n = 128, float: 20 us of
  // 65; n = 100, bfloat16: 22 of 102).  (Rows past n arrive as zeros; an odd n in bfloat16 has rows that are not whole dwords.)
  reg w[CG * (kPer == 1 ? 64 : 16)];
  {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    constexpr int kQuads = kPer == 1 ? 4 : 2, kUnits = 16 / kQuads;            // loads of a gate's 16 units, units in one
    const __amdgpu_buffer_rsrc_t rs = frame_of(d.W, (unsigned)(4 * n * n * sizeof(T)));
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      const int out = cg * 64 + lane;
      unsigned v[64];                                                          // [gate][unit]
      if (kPer == 1 || n % 2 == 0) {
        u32x4 x[4 * kQuads];
#pragma unroll
        for (int i = 0; i < 4 * kQuads; ++i)
          x[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)((out * 4 * n + i / kQuads * n + wave * 16 + i % kQuads * kUnits) * sizeof(T)), 0, 0);
#pragma unroll
        for (int i = 0; i < 64; ++i) {
          const int e = i % kUnits;
          if constexpr (kPer == 1) v[i] = x[i / kUnits][e];
          else v[i] = (e & 1) ? x[i / kUnits][e >> 1] >> 16 : x[i / kUnits][e >> 1] & 0xffffu;
        }
      } else {
        const uint16_t* W = (const uint16_t*)d.W + (long)min(out, n - 1) * 4 * n;
#pragma unroll
        for (int i = 0; i < 64; ++i) v[i] = W[(i >> 4) * n + min(wave * 16 + (i & 15), n - 1)];
#pragma unroll
        for (int i = 0; i < 64; ++i) { all_in_flight(v[i]); v[i] = out < n ? v[i] : 0u; }
      }
#pragma unroll
      for (int i = 0; i < 64; ++i) v[i] = wave * 16 + (i & 15) < n ? v[i] : 0u;
      if constexpr (kPer == 1) {
#pragma unroll
        for (int i = 0; i < 64; ++i) w[cg * 64 + i] = __uint_as_float(v[i]);
      } else {
#pragma unroll
        for (int bk = 0; bk < 16; ++bk) w[cg * 16 + bk] = (u32x2){v[bk] | (v[16 + bk] << 16), v[32 + bk] | (v[48 + bk] << 16)};
      }
    }
  }
  // the error word (nothing here waits for another work-group) and the counters of the products behind this loop (gemm_tiny.hip)
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.sync = 0u;
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = tid; i < a.ncounters; i += 64 * NW) a.counters[i] = 0u;
  const int L = !active ? 0 : a.lens ? max(0, min((int)len_bits, Tn)) : Tn;
  // What the gate gradients take from a frame's inputs alone: dc = Dc + dh f_c, Dc' = dc gf, dz = (dc f_i, dc f_f, dc f_g, dh f_o), dh = dy + Dh
  // (lstm_cell_grad has the plain form; the factors are multiplied in another order here, with as many roundings, so last places differ).  The inputs are taken, and tanh of the state, behind the products of the step before; the rest
  // goes where the compiler finds room, the read of the shares of Dh among it.  (Taken by moves that it cannot put off: what it does with a place that
  // is being loaded again is waited for together with all that has been asked for since.)
  struct { float gi, gf, gg, go, c_prev, dy, tc; bool valid; } x;
  int t = (int)last;                                                           // frame of the step whose inputs are taken next
  auto moved = [](float v) __attribute__((always_inline)) { float o; asm volatile("v_mov_b32 %0, %1" : "=v"(o) : "v"(v)); return o; };
  auto take = [&](const In& v) __attribute__((always_inline)) {
    x.tc = tanhf_(c_new);
    asm volatile("" : "+v"(x.tc));
    x.valid = t < L;                                                           // (L is 0 in lanes without a cell)
    x.gi = moved(v.gi); x.gf = moved(v.gf); x.gg = moved(v.gg); x.go = moved(v.go);
    x.c_prev = moved(v.c_prev);
    x.dy = moved(kPer == 1 ? __uint_as_float(v.dy_bits) : __uint_as_float((unsigned)v.dy_bits << 16));
    c_new = x.c_prev;
    t += d.rev ? 1 : -1;
  };
  // Dh of the rows that had a frame in the last step: the wavefronts' shares
  auto collect = [&](int buf, bool take, auto&& meanwhile) __attribute__((always_inline)) {
    float v[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) v[k] = red[buf][k][u >> 6][u & 63][r];
    __builtin_amdgcn_sched_barrier(0);
    meanwhile();
    float sum = v[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) sum += v[k];
    Dh = take ? sum : Dh;
  };

  take(in[0]);
  bool had = false;
  auto step = [&](int, auto S) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
    const float f_c = x.go * (1.f - x.tc * x.tc), f_i = x.gg * x.gi * (1.f - x.gi), f_f = x.c_prev * x.gf * (1.f - x.gf);
    const float f_g = x.gi * (1.f - x.gg * x.gg), f_o = x.tc * x.go * (1.f - x.go);
    collect((s & 1) ^ 1, had, [&]() __attribute__((always_inline)) { fetch(in[s]); });       // (in the first step there is nothing to take)
    had = x.valid;
    const float dh = x.dy + Dh, dc = Dc + dh * f_c;
    float dz[4] = {dc * f_i, dc * f_f, dc * f_g, dh * f_o};
    Dc = x.valid ? dc * x.gf : Dc;
#pragma unroll
    for (int q = 0; q < 4; ++q) dz[q] = x.valid ? dz[q] : 0.f;
    const u32x2 bits = {pack_bf16x2(dz[0], dz[1]), pack_bf16x2(dz[2], dz[3])};
    f32x4 acc[CG][2];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[cg][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // a fourth of the products: blocks of units bk, bk + 4, ... of the wavefront's sixteen
    auto products = [&](auto Part) __attribute__((always_inline)) {
      constexpr int part = decltype(Part)::value;
      static_for<4>([&](auto Bk) __attribute__((always_inline)) {
        constexpr int bk = 4 * part + decltype(Bk)::value;
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          if constexpr (kPer == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[cg][q & 1] = mma4<bk>(dz[q], w[(cg * 4 + q) * 16 + bk], acc[cg][q & 1]);
          } else {
            acc[cg][bk & 1] = mma4<bk>(bits, w[cg * 16 + bk], acc[cg][bk & 1]);
          }
        }
      });
    };
    products(std::integral_constant<int, 0>{});
    products(std::integral_constant<int, 1>{});
    {
      const __amdgpu_buffer_rsrc_t rz = frame_of(z_out, z_bytes);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (kPer == 1) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dz[q]), rz, z_off, q * z_gate, 0);
        else __builtin_amdgcn_raw_buffer_store_b16((unsigned short)((q & 1) ? bits[q >> 1] >> 16 : bits[q >> 1]), rz, z_off, q * z_gate, 0);
        dbsum[q] += dz[q];
      }
      z_out += z_step;
    }
    products(std::integral_constant<int, 2>{});
    take(in[(s + 1) % kAhead]);
    products(std::integral_constant<int, 3>{});
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) *(f32x4*)&red[s & 1][wave][cg][lane][0] = acc[cg][0] + acc[cg][1];
    meet();
  };
  if (Tn > 0) {
    walk(Tn, step);
    collect((Tn - 1) & 1, had, [] {});
  }
  if (active) {
    if (d.dh0) d.dh0[(long)b * n + u] = Dh;
    if (d.dc0) d.dc0[(long)b * n + u] = Dc;
  }
  // bias gradient: the four rows of this work-group; into its slice, or, if it is the only one, straight to its place
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float s = dbsum[q];
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
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
