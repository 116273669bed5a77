// Single-launch loops of wide layers (bfloat16, 1024 < n <= 2048): W_h in blocks over the whole device.
//
// The kernels of persistent.hip give a work-group all of K for its units, which is twice the registers of a compute unit here, and
// the per-step kernels read all 32 MB of W_h again in every step (n = 2048: 11 us forward, 22 backward).  Here
// work-group (i, j) holds a block of W_h with all four gates - 128 registers of a lane - for all 32 rows of a slab, and
// a step is two exchanges, each of far less data than one exchange of the other shape would be:
//   forward    (i, j) multiplies h of range i (512 units) for the 32 units of column j, publishes its share of z; the members of column j (a task
//              of eight rows each) add the shares, do the cell and publish h.  (Blocks of 128 x 128 units as below publish 16 MB of shares a step.)
//   backward   (i, j) multiplies dz of block i (128 units) by W_h^T, publishes its share of Dh for block j; the members of column j add the shares, do
//              the gate gradients and publish dz
// Shares stay inside column j, whose members are placed on one XCD; h and dz go to row j of the grid, across XCDs.
//
// Exchange as in persistent.hip: two slots per ring, and in every 8 bytes a tag bit - bit 30 of the second dword - of the step that wrote
// them; 16 bytes of a share are four rows of one column, 8 of h or dz four units of one row.  Values that travel are scaled by 2^-32 where
// they are not bounded by 1 (shares, dz), which leaves that bit free below 2^32.  What is not in that range, NaN and infinities included, arrives all the same:
//   shares  folded into the patterns between 1 and 2 (exchange_dev.h), in a second store that corrects the first;
//   h       is bounded or NaN: a NaN in the tagged unit goes into its untagged neighbours of the same row, every product with that row is NaN either way;
//   dz      has no patterns to spare in 16 bits: the tagged unit says "wide", and the reader fetches the row's values from DZ, which their
//           writer has stored and released before it published.
// (Looking for such values costs 0.15 us of a backward step, 4.33 -> 4.48 us, and nothing forward, 4.04 -> 3.94.)
// Sums are taken in the order of the producers.
// A slot may be written again because its readers have had to finish with it: h of step s + 2 needs shares of step s + 1 from column j,
// those need h of step s + 1 from every block, and that needs the shares of step s from every work-group; likewise for the shares and backward.
//
// What bounds a step is the two exchanges, about 0.8 us for shares and 1.4 for h or dz, not the product (0.8 us, half of it operand reads from LDS).
// Measured at n = 2048, 32 rows, 140 steps, the kernels alone: 3.9 us a step forward and 4.5 backward; 11.1 and 21.9 in the per-step kernels.
#include "exchange_dev.h"
#include <algorithm>

namespace lstm {
namespace {

constexpr int kBlk = 128, kSlab = 32;
constexpr float kScale = 1.f / 4294967296.f;              // 2^-32
constexpr unsigned kTagBit = 1u << 30;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const char* p) { return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)0x7ff00000, kBufFlags); }
constexpr unsigned kParked = 0x7ff00000u;                 // an offset outside every descriptor: reads zero, writes nothing
constexpr int kNt = 2;                                    // cache policy: non-temporal
// Frame t of an array, so that a lane's offset inside a frame is all a step needs: no lane computes an address, none branches.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frame(const void* base, long t, long frame_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + t * frame_bytes), 0, base ? (int)kParked : 0, kBufFlags);
}
__device__ __forceinline__ float ldf(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, soff, kNt)); }
__device__ __forceinline__ void stf(float v, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned soff) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, off, soff, kNt); }
__device__ __forceinline__ unsigned tag_of(int step) { return ll_fwd_tag((unsigned)step) << 30; }

// Fetches N 16-byte pieces per lane, 4 KiB apart, until the first `count` (uniform) carry `tag` in both halves (bounded); the others read as zeros.
// The first piece is asked for alone until it has turned: all of them in every poll would be 8 MB of reads a round.  No load is predicated
// (what lies behind the pieces is ring memory too): with a branch per load the compiler waited for each before the next, 3.7 us instead of 1.
// wide(x) is called when all tags have turned and some lane's tagged dwords, tags off, hold something of 1 or more in magnitude; it returns
// whether x, changed by it, will do.  Looked at together with the tags: a branch of its own on every step's way cost 0.04 us.
template <bool WIDE, int N, typename F>
__device__ __forceinline__ void await_pieces(u32x4 (&x)[N], int count, __amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned slot, unsigned tag, bool& dead,
                                             unsigned* err, unsigned limit, F&& wide) {
  const auto differs = [&](const u32x4& v) { return (v[1] ^ tag) | (v[3] ^ tag); };
  // With the tag still in it a dword of 1 or more in magnitude reads as that, or, if the tag is set, as infinity or NaN.
  const float one = __uint_as_float(kOneBits | tag);
  unsigned clear = ~kTagBit;
  for (unsigned poll = 0, first = 1; !dead && count > 0; ++poll) {
    if (first) {
      if (__builtin_amdgcn_ballot_w64((differs(__builtin_amdgcn_raw_buffer_load_b128(rs, voff, slot, kSc1)) & kTagBit) != 0u) == 0ull) { first = 0; continue; }
    } else {
#pragma unroll
      for (int it = 0; it < N; ++it) x[it] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, slot + it * 4096u, kSc1);
      unsigned bits = 0u;
#pragma unroll
      for (int it = 0; it < N; ++it) bits |= differs(x[it]) & (it < count ? kTagBit : 0u);
      float m[2] = {0.f, 0.f};
#pragma unroll
      for (int it = 0; it < N && WIDE; ++it) m[it & 1] = max_magnitude(m[it & 1], __uint_as_float(x[it][1]), __uint_as_float(x[it][3]));
      const bool big = WIDE && !(max_magnitude(0.f, m[0], m[1]) < one);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64((bits != 0u) | big) == 0ull, 1)) break;
      if (WIDE && __builtin_amdgcn_ballot_w64(bits != 0u) == 0ull) {
#pragma unroll
        for (int it = 0; it < N; ++it) { x[it][1] &= ~kTagBit; x[it][3] &= ~kTagBit; }
        if (wide(x)) { clear = ~0u; break; }
      }
    }
    if (poll >= limit || ((poll & 63u) == 63u && ld_relaxed(err) != 0u)) {
      st_relaxed(err, 1u);
      dead = true;
    }
  }
#pragma unroll
  for (int it = 0; it < N; ++it) {
    const unsigned keep = it < count && !dead ? ~0u : 0u;
    x[it] = (u32x4){x[it][0] & keep, x[it][1] & keep & clear, x[it][2] & keep, x[it][3] & keep & clear};
  }
}
// Shares in: folded ones unfolded; where one of them only says that it follows, the pieces are fetched again.
__device__ __forceinline__ void await_shares(u32x4 (&x)[4], int count, __amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned slot, unsigned tag, bool& dead,
                                             unsigned* err, unsigned limit) {
  await_pieces<true>(x, count, rs, voff, slot, tag, dead, err, limit, [&](u32x4 (&v)[4]) {
    bool follows = false;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      follows |= it < count && ((v[it][1] & 0x7fffffffu) == kOneBits || (v[it][3] & 0x7fffffffu) == kOneBits);
      v[it][1] = unfold_wide(v[it][1]);
      v[it][3] = unfold_wide(v[it][3]);
    }
    return __builtin_amdgcn_ballot_w64(follows) == 0ull;
  });
}
// Shares out: clamped to 1, which is nothing to wait for, and looked at behind the stores.
template <int NRT>
__device__ __forceinline__ void publish_shares(f32x4 (&acc)[NRT][2], __amdgpu_buffer_rsrc_t rs, const unsigned (&off)[NRT], unsigned slot, unsigned tag,
                                               int local) {
  const auto store = [&](auto&& on_wire) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) {
        const f32x4& a = acc[rt][ct];
        const u32x4 v = {__float_as_uint(a[0]), on_wire(a[1]) | tag, __float_as_uint(a[2]), on_wire(a[3]) | tag};
        if (local) __builtin_amdgcn_raw_buffer_store_b128(v, rs, off[rt], slot + ct * 256u, 1);
        else __builtin_amdgcn_raw_buffer_store_b128(v, rs, off[rt], slot + ct * 256u, 16);
      }
  };
  store([](float v) { return __float_as_uint(__builtin_amdgcn_fmed3f(v, -1.f, 1.f)); });       // (NaN: -1)
  float m = 0.f;
#pragma unroll
  for (int f = 0; f < 2 * NRT; ++f) m = max_magnitude(m, acc[f >> 1][f & 1][1], acc[f >> 1][f & 1][3]);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(is_wide(m)) != 0ull, 0)) store([](float v) { return fold_wide(__float_as_uint(v)); });
}
// Four neighbouring lanes' 16 bits in the first of them (the others get something else), tagged.  H: a tagged value
// that does not leave its bit free is NaN, and makes the two beside it NaN.
template <bool H>
__device__ __forceinline__ u32x2 four_lanes(unsigned x0, unsigned tag) {
  const unsigned x1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x101, 0xf, 0xf, true);
  const unsigned x2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x102, 0xf, 0xf, true);
  const unsigned x3 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x103, 0xf, 0xf, true);
  const unsigned nan = H ? (unsigned)((int)(x3 << 17) >> 31) : 0u;     // bit 14
  return (u32x2){x0 | (x1 << 16) | nan, ((x2 | (x3 << 16)) & ~kTagBit) | tag};
}
__device__ __forceinline__ f32x4 mma(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Both kernels end a step's product with operands in LDS, every wavefront wanting all of them: 16 chunks x NRT row tiles, two column tiles of its own.
template <int NRT>
__device__ __forceinline__ void product(f32x4 (&acc)[NRT][2], const u32x4* zs, const u32x4 (&w)[2][16], int lane) {
  constexpr int kAll = 16 * NRT, kWin = 8;                 // operand reads in flight (fenced: left alone the compiler moves each down to its use and waits there)
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) acc[rt][0] = acc[rt][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
  u32x4 av[kWin];
#pragma unroll
  for (int p = 0; p < kWin; ++p) av[p] = zs[p * 64 + lane];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < kAll; ++p) {
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[p % NRT][c] = mma(av[p % kWin], w[c][p / NRT], acc[p % NRT][c]);
    if (p + kWin < kAll) av[p % kWin] = zs[(p + kWin) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ---- forward: column j = units 32 j .. + 31, K range i = `cb` chunks of 32 units; wavefront = gate.  A task is eight rows of column j.
template <int NRT>
__global__ __launch_bounds__(256) void block_fwd_kernel(BlockFwdArgs a) {
  __shared__ u32x4 zs[16 * NRT * 64];
  __shared__ float zb[2][8][4][33];                        // [task][row][gate][unit]
  const int n = a.n, B = a.B, Tn = a.T, J = (n + 31) / 32, I = a.ni, cb = (J + I - 1) / I;
  const int slot_ = blockIdx.x >> 3;
  const int i = __builtin_amdgcn_readfirstlane(slot_ % I), j = __builtin_amdgcn_readfirstlane((slot_ / I) * 8 + (blockIdx.x & 7));     // column j on one XCD
  if (j >= J) return;
  publish_xcd(a.xcc, j * I, i);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned h_slot = 64u * 2048u, part_slot = (unsigned)J * 4u * 4u * 4096u;
  bool dead = false;

  u32x4 w[2][16];
  {
    const u32x4* src = (const u32x4*)a.W + (((long)j * I + i) * 4 + wave) * 2 * 16 * 64 + lane;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int ch = 0; ch < 16; ++ch) w[c][ch] = src[(c * 16 + ch) * 64];
  }
  const int my_chunks = max(0, min(cb, J - i * cb));       // (the last range may be shorter; what is missing is zeros)
  const int h_pieces = (my_chunks * NRT - wave + 3) / 4;
  // Rows use h0 - from memory, it need not be bounded by 1 - up to their first frame.
  int last_start = 0;
  for (int b = a.row0; b < min(B, a.row0 + 16 * NRT) && a.rev && a.lens; ++b) last_start = max(last_start, Tn - clamp_len(a.lens, b, Tn));
  const int local = group_is_xcd_local(a.xcc, j * I, I, a.spin_limit);

  // tasks i and i + I; thread = (row, unit)
  const int r8 = tid >> 5, u = j * 32 + (tid & 31);
  bool on[2], active[2], started[2] = {false, false};
  int b[2], L[2];
  float c[2] = {0.f, 0.f}, h[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    on[k] = i + k * I < 2 * NRT;
    b[k] = a.row0 + 8 * (i + k * I) + r8;
    active[k] = on[k] && b[k] < B && u < n;
    if (!active[k]) b[k] = 0;
    L[k] = active[k] ? clamp_len(a.lens, b[k], Tn) : 0;
    if (active[k]) {
      if (a.c0) c[k] = a.c0[(long)b[k] * n + u];
      if (a.h0) h[k] = a.h0[(long)b[k] * n + u];
    }
  }
  const long g_frame = (long)B * 4 * n * 4;
  const __amdgpu_buffer_rsrc_t h_rs = rsrc(a.ring), p_rs = rsrc(a.ring + 2 * h_slot);
  const unsigned h_in = (unsigned)(i * cb) * NRT * 1024u + tid * 16u;
  unsigned h_out[2], p_in[2], p_out[NRT];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int row = 8 * (i + k * I) + r8, u32 = tid & 31;  // row of the slab; ring [chunk][row tile][lane] x 16
    h_out[k] = (lane & 3) == 0 ? (unsigned)(((j * NRT + (row >> 4)) * 64 + (u32 >> 3) * 16 + (row & 15)) * 16 + ((u32 >> 2) & 1) * 8) : kParked;
    p_in[k] = (unsigned)((j * 4 + i + k * I) * I) * 4096u + tid * 16u;
  }
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {                       // rows 4 (lane / 16) .. of the row tile: half a task
    const int quad = rt * 4 + (lane >> 4);
    p_out[rt] = (unsigned)((j * 4 + (quad >> 1)) * I + i) * 4096u + (unsigned)((quad & 1) * 128 + wave * 32 + (lane & 15)) * 16u;
  }
  float zx[2][4];
  auto fetch = [&](int tau) __attribute__((always_inline)) {
    const int t = a.rev ? Tn - 1 - tau : tau;
    const __amdgpu_buffer_rsrc_t rs = frame(a.gates, t, g_frame);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      const unsigned off = t < L[k] ? (unsigned)(b[k] * 4 * n + u) * 4u : kParked;
#pragma unroll
      for (int q = 0; q < 4; ++q) zx[k][q] = ldf(rs, off, (unsigned)(q * n) * 4u);
    }
  };
  fetch(0);

  for (int tau = 0; tau < Tn; ++tau) {
    const int t = a.rev ? Tn - 1 - tau : tau;
    const unsigned tag = tag_of(tau), p_slot = (tau & 1) * part_slot;
    {                                                      // h of this range, into LDS
      u32x4 x[4 * NRT];
      if (tau > 0) await_pieces<false>(x, h_pieces, h_rs, h_in, ((tau - 1) & 1) * h_slot, tag_of(tau - 1), dead, a.sync, a.spin_limit, [](auto&) { return true; });
      else {
#pragma unroll
        for (int p = 0; p < 4 * NRT; ++p) x[p] = (u32x4){0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int p = 0; p < 4 * NRT; ++p) zs[p * 256 + tid] = x[p];
#pragma unroll 1
      for (int p = 0; p < 4 * NRT && tau <= last_start; ++p) {
        const int piece = p * 4 + wave, ch = piece / NRT, row = a.row0 + (piece % NRT) * 16 + (lane & 15);
        const int k0 = (i * cb + ch) * 32 + (lane >> 4) * 8;
        if (row >= B || ch >= my_chunks || tau > (a.rev ? Tn - clamp_len(a.lens, row, Tn) : 0)) continue;
        u32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = a.h0 && k0 + 2 * e < n ? a.h0[(long)row * n + k0 + 2 * e] : 0.f;
          const float hi = a.h0 && k0 + 2 * e + 1 < n ? a.h0[(long)row * n + k0 + 2 * e + 1] : 0.f;
          v[e] = f2bf_bits(lo) | ((unsigned)f2bf_bits(hi) << 16);
        }
        zs[p * 256 + tid] = v;
      }
    }
    __syncthreads();
    f32x4 acc[NRT][2];
    product<NRT>(acc, zs, w, lane);
    publish_shares<NRT>(acc, p_rs, p_out, p_slot, tag, local);
    // the shares of this work-group's tasks: thread = (half of the rows, gate, unit), four rows
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      u32x4 x[4];
      await_shares(x, I, p_rs, p_in[k], p_slot, tag, dead, a.sync, a.spin_limit);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        zb[k][4 * (tid >> 7) + v][(tid >> 5) & 3][tid & 31] =
            ((__uint_as_float(x[0][v]) + __uint_as_float(x[1][v])) + (__uint_as_float(x[2][v]) + __uint_as_float(x[3][v]))) * (1.f / kScale);
    }
    __syncthreads();                                       // (zb is written again behind the next step's first barrier)
    CellOut o[2] = {};
    float h_before[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      const float zh[4] = {zb[k][r8][0][tid & 31], zb[k][r8][1][tid & 31], zb[k][r8][2][tid & 31], zb[k][r8][3][tid & 31]};
      h_before[k] = h[k];
      if (t < L[k]) {
        o[k] = lstm_cell(zh, zx[k], c[k]);
        c[k] = o[k].c; h[k] = o[k].h; started[k] = true;
      }
      __builtin_amdgcn_raw_buffer_store_b64(four_lanes<true>(started[k] ? f2bf_bits(h[k]) : 0u, tag), h_rs, h_out[k], (tau & 1) * h_slot, 16);
    }
    const __amdgpu_buffer_rsrc_t y_rs = frame(a.y, t, (long)B * a.ldy * 2), hp_rs = frame(a.hprev, t, (long)B * a.ldh * 2), c_rs = frame(a.cs, t, (long)B * n * 4),
                                 g_rs = frame(a.gates, t, g_frame);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      const bool valid = t < L[k];
      const unsigned g_off = valid && a.write_gates ? (unsigned)(b[k] * 4 * n + u) * 4u : kParked;
      __builtin_amdgcn_raw_buffer_store_b16(valid ? f2bf_bits(h[k]) : (uint16_t)0, y_rs, active[k] ? (unsigned)(b[k] * a.ldy + u) * 2u : kParked, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b16(f2bf_bits(h_before[k]), hp_rs, active[k] ? (unsigned)(b[k] * a.ldh + u) * 2u : kParked, 0, 0);
      stf(c[k], c_rs, active[k] ? (unsigned)(b[k] * n + u) * 4u : kParked, 0);
      stf(o[k].gi, g_rs, g_off, 0); stf(o[k].gf, g_rs, g_off, (unsigned)n * 4u);
      stf(o[k].gg, g_rs, g_off, (unsigned)n * 8u); stf(o[k].go, g_rs, g_off, (unsigned)n * 12u);
    }
    if (tau + 1 < Tn) fetch(tau + 1);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (active[k]) {
      if (a.hT) a.hT[(long)b[k] * n + u] = h[k];
      if (a.cT) a.cT[(long)b[k] * n + u] = c[k];
    }
}

// ---- backward: blocks of 128 units.  A task of column j: rows 4 quad .. + 3 of the slab, units j * 128 + 64 half .. + 63; thread = (row, unit).
template <int NRT>
__global__ __launch_bounds__(256) void block_bwd_kernel(BlockBwdArgs a) {
  __shared__ u32x4 zs[16 * NRT * 64];                      // dz of block i: [chunk][row tile][lane]
  __shared__ float red[2][4][4][66];                       // [task][wavefront][row][unit]
  constexpr int kQuads = 4 * NRT;
  const int n = a.n, B = a.B, Tn = a.T, nb = (n + kBlk - 1) / kBlk;
  // column j (its nb members i) on one XCD: XCD x runs columns 2x and 2x + 1
  const int slot_ = blockIdx.x >> 3, second = slot_ >= nb;
  const int j = __builtin_amdgcn_readfirstlane(2 * (blockIdx.x & 7) + second), i = __builtin_amdgcn_readfirstlane(slot_ - second * nb);
  if (j >= nb) return;
  publish_xcd(a.xcc, j * nb, i);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned dz_slot = (unsigned)nb * 32768u, part_slot = (unsigned)nb * nb * 16u * 1024u;
  bool dead = false;

  u32x4 w[2][16];                                          // [column tile][chunk]: outputs j * 128 + (2 wave + c) * 16 + lane % 16, straight from rows of W_h
  if (n % 8 == 0) {                                        // (all loads in flight: addresses clamped, what they fetch then masked)
#pragma unroll
    for (int f = 0; f < 32; ++f) {
      const int out = j * kBlk + (2 * wave + (f >> 4)) * 16 + (lane & 15), u0 = i * kBlk + (f & 3) * 32 + (lane >> 4) * 8;
      w[f >> 4][f & 15] = *(const u32x4*)((const uint16_t*)a.W + (long)min(out, n - 1) * 4 * n + ((f >> 2) & 3) * n + min(u0, n - 8));
      if (out >= n || u0 >= n) w[f >> 4][f & 15] = (u32x4){0u, 0u, 0u, 0u};
    }
  } else {
#pragma unroll
    for (int f = 0; f < 32; ++f) {
      const int out = j * kBlk + (2 * wave + (f >> 4)) * 16 + (lane & 15), u0 = i * kBlk + (f & 3) * 32 + (lane >> 4) * 8;
      const uint16_t* p = (const uint16_t*)a.W + (long)min(out, n - 1) * 4 * n + ((f >> 2) & 3) * n;
      unsigned e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) { e[k] = p[min(u0 + k, n - 1)]; if (out >= n || u0 + k >= n) e[k] = 0u; }
      w[f >> 4][f & 15] = (u32x4){e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
  }
  const int local = group_is_xcd_local(a.xcc, j * nb, nb, a.spin_limit);

  bool on[2], active[2];
  int b[2], u[2], L[2], quad[2];
  float Dh[2] = {0.f, 0.f}, Dc[2] = {0.f, 0.f}, dbsum[2][4] = {};
  const __amdgpu_buffer_rsrc_t z_rs = rsrc(a.ring), p_rs = rsrc(a.ring + 2 * dz_slot);
  unsigned z_out[2], p_in[2], p_out[NRT];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int task = i + k * nb;
    on[k] = task < 2 * kQuads;
    quad[k] = task % kQuads;
    const int half = (task / kQuads) & 1, row = 4 * quad[k] + wave, u32 = lane & 31;
    b[k] = a.row0 + row;
    u[k] = j * kBlk + 64 * half + lane;
    active[k] = on[k] && b[k] < B && u[k] < n;
    if (!active[k]) b[k] = 0;
    L[k] = active[k] ? clamp_len(a.lens, b[k], Tn) : 0;
    if (active[k]) {
      if (a.dhT) Dh[k] = a.dhT[(long)b[k] * n + u[k]];
      if (a.dcT) Dc[k] = a.dcT[(long)b[k] * n + u[k]];
    }
    // ring [block][chunk = 4 gate + unit / 32][row tile][lane] x 16
    z_out[k] = (lane & 3) == 0 ? (unsigned)((((j * 16 + 2 * half + (lane >> 5)) * NRT + (row >> 4)) * 64 + (u32 >> 3) * 16 + (row & 15)) * 16 + ((u32 >> 2) & 1) * 8)
                               : kParked;
    p_in[k] = (unsigned)((j * 16 + task) * nb + wave) * 1024u + lane * 16u;
  }
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt)
    p_out[rt] = (unsigned)((j * 16 + rt * 4 + (lane >> 4) + kQuads * (wave >> 1)) * nb + i) * 1024u + (unsigned)((2 * wave & 3) * 16 + (lane & 15)) * 16u;
  const long g_frame = (long)B * 4 * n * 4, s_frame = (long)B * n * 4;
  float gi[2], gf[2], gg[2], go[2], c_new[2], c_prev[2];
  uint16_t dy[2];                                          // (converted where it is used: that is what waits for the load)
  auto fetch = [&](int sigma) __attribute__((always_inline)) {
    const int tau = Tn - 1 - sigma, t = a.rev ? Tn - 1 - tau : tau, t_prev = a.rev ? t + 1 : t - 1;
    const bool inside = t_prev >= 0 && t_prev < Tn;
    const __amdgpu_buffer_rsrc_t g_rs = frame(a.gates, t, g_frame), c_rs = frame(a.cs, t, s_frame), p_rs = frame(inside ? a.cs : a.c0, inside ? t_prev : 0, s_frame),
                                 y_rs = frame(a.dy, t, (long)B * a.lddy * 2);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      const bool valid = t < L[k];
      const unsigned g_off = valid ? (unsigned)(b[k] * 4 * n + u[k]) * 4u : kParked, s_off = valid ? (unsigned)(b[k] * n + u[k]) * 4u : kParked;
      gi[k] = ldf(g_rs, g_off, 0); gf[k] = ldf(g_rs, g_off, (unsigned)n * 4u);
      gg[k] = ldf(g_rs, g_off, (unsigned)n * 8u); go[k] = ldf(g_rs, g_off, (unsigned)n * 12u);
      c_new[k] = ldf(c_rs, s_off, 0);
      c_prev[k] = ldf(p_rs, s_off, 0);
      dy[k] = __builtin_amdgcn_raw_buffer_load_b16(y_rs, valid ? (unsigned)(b[k] * a.lddy + u[k]) * 2u : kParked, 0, 0);
    }
  };
  fetch(0);

  for (int sigma = 0; sigma <= Tn; ++sigma) {              // step Tn only collects the Dh that leaves the layer
    const int tau = Tn - 1 - sigma;
    const int t = a.rev ? Tn - 1 - tau : tau, t_next = a.rev ? t - 1 : t + 1;
    const unsigned tag = tag_of(sigma), z_slot = (sigma & 1) * dz_slot, p_slot = (sigma & 1) * part_slot;
    if (sigma > 0) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (!on[k]) continue;
        u32x4 x[4];                                        // producers wave, wave + 4, ...
        await_shares(x, (nb - wave + 3) / 4, p_rs, p_in[k], part_slot - p_slot, tag_of(sigma - 1), dead, a.sync, a.spin_limit);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          red[k][wave][v][lane] = (__uint_as_float(x[0][v]) + __uint_as_float(x[1][v])) + (__uint_as_float(x[2][v]) + __uint_as_float(x[3][v]));
      }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t d_rs = frame(a.DZ, sigma == Tn ? 0 : t, g_frame / 2);
    float dz[2][4] = {};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
      if (sigma > 0 && t_next >= 0 && t_next < L[k])
        Dh[k] = ((red[k][0][wave][lane] + red[k][1][wave][lane]) + (red[k][2][wave][lane] + red[k][3][wave][lane])) * (1.f / kScale);
      if (sigma == Tn) continue;
      if (t < L[k]) lstm_cell_grad(gi[k], gf[k], gg[k], go[k], c_new[k], c_prev[k], bf_bits2f(dy[k]) + Dh[k], Dc[k], dz[k]);
      float v[4];
      unsigned x[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {                        // (scaled by a power of two: exact)
        v[g] = bf_bits2f(f2bf_bits(dz[k][g])) * kScale;
        x[g] = __float_as_uint(v[g]) >> 16;
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(is_wide(max_magnitude(max_magnitude(0.f, v[0], v[1]), v[2], v[3]))) != 0ull, 0)) {
        const unsigned off = active[k] ? (unsigned)(b[k] * 4 * n + u[k]) * 2u : kParked;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          __builtin_amdgcn_raw_buffer_store_b16(f2bf_bits(dz[k][g]), d_rs, off, (unsigned)(g * n) * 2u, 16);
          if ((lane & 3) == 3 && (x[g] & 0x7fffu) >= 0x3f80u) x[g] = 0x3f80u;        // "wide": 1 in magnitude
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) __builtin_amdgcn_raw_buffer_store_b64(four_lanes<false>(x[g], tag), z_rs, z_out[k], z_slot + g * (4 * NRT * 1024u), 16);
    }
    if (sigma == Tn) break;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!on[k]) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g) dbsum[k][g] += dz[k][g];
      const unsigned off = active[k] ? (unsigned)(b[k] * 4 * n + u[k]) * 2u : kParked;
#pragma unroll
      for (int g = 0; g < 4; ++g) __builtin_amdgcn_raw_buffer_store_b16(f2bf_bits(dz[k][g]), d_rs, off, (unsigned)(g * n) * 2u, 0);
    }
    if (sigma + 1 < Tn) fetch(sigma + 1);
    {                                                      // dz of block i, into LDS
      u32x4 x[4 * NRT];
      await_pieces<true>(x, 4 * NRT, z_rs, (unsigned)i * (16u * NRT * 1024u) + tid * 16u, z_slot, tag, dead, a.sync, a.spin_limit, [&](u32x4 (&v)[4 * NRT]) {
        // values that the ring cannot hold: from DZ, eight units of a row and gate
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        int at = lane;                                     // (opaque: what is computed from it stays in here instead of in registers all the way)
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int p = 0; p < 4 * NRT; ++p) {
          if (!is_wide(max_magnitude(0.f, __uint_as_float(v[p][1]), __uint_as_float(v[p][3])))) continue;
          const int piece = p * 4 + wave, ch = piece / NRT, row = a.row0 + (piece % NRT) * 16 + (at & 15), u0 = i * kBlk + (ch & 3) * 32 + (at >> 4) * 8;
          unsigned e[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const unsigned off = row < B && u0 + k < n ? (unsigned)((row * 4 + (ch >> 2)) * n + u0 + k) * 2u : kParked;
            e[k] = __float_as_uint(bf_bits2f(__builtin_amdgcn_raw_buffer_load_b16(d_rs, off, 0, kSc1)) * kScale) >> 16;
          }
          v[p] = (u32x4){e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
        return true;
      });
#pragma unroll
      for (int p = 0; p < 4 * NRT; ++p) zs[p * 256 + tid] = x[p];
    }
    __syncthreads();
    f32x4 acc[NRT][2];
    product<NRT>(acc, zs, w, lane);
    publish_shares<NRT>(acc, p_rs, p_out, p_slot, tag, local);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (active[k]) {
      if (a.dh0) a.dh0[(long)b[k] * n + u[k]] = Dh[k];
      if (a.dc0) a.dc0[(long)b[k] * n + u[k]] = Dc[k];
    }
    if (!a.dbpart || !on[k]) continue;                     // bias gradient: a slice per four rows
#pragma unroll
    for (int g = 0; g < 4; ++g) red[k][wave][g][lane] = dbsum[k][g];
    __syncthreads();
    if (u[k] < n)
      a.dbpart[(long)(a.row0 / 4 + quad[k]) * 4 * n + wave * n + u[k]] =
          (red[k][0][wave][lane] + red[k][1][wave][lane]) + (red[k][2][wave][lane] + red[k][3][wave][lane]);
  }
}

// Forward W_h: [j][i][gate][column tile][chunk][lane] x 16 bytes, scaled by 2^-32.  Thread = (eight k, eight units of a gate): 16-byte reads of eight
// rows, the 8 x 8 block turned in registers (n = 2048: 23 us, 31 with two-byte reads and a turn through LDS).
// Blocks from row `packs` on clear what the loop behind it wants cleared (a launch of its own: two layers of n = 2048, 32 rows, 1043 us a training pass, now 1036).
__global__ __launch_bounds__(256) void pack_blocks_kernel(const bf16_t* W_, uint4* out, int n, int I, ZeroRegions z, int packs) {
  if ((int)blockIdx.y >= packs) {
    const int block = (blockIdx.y - packs) * gridDim.x + blockIdx.x;
    if (block < z.first_block[z.count]) fill_zero_body(z, block, threadIdx.x);
    return;
  }
  const int J = (n + 31) / 32, cb = (J + I - 1) / I;
  const int lo = threadIdx.x & 7, gate = (threadIdx.x >> 3) & 3, k8 = (threadIdx.x >> 5) & 7;      // a block: 64 units, 64 k, the four gates
  const int kk = blockIdx.x * 8 + k8, u8 = blockIdx.y * 8 + lo, u0 = u8 * 8;                       // kk: eights of k, counted through the ranges (16 chunks each)
  const int i = kk / 64, ch = (kk / 4) % 16, k0 = (i * cb + ch) * 32 + (kk & 3) * 8, j = u8 >> 2;
  if (j >= J) return;
  const uint16_t* p = (const uint16_t*)W_ + gate * n;
  unsigned r[8][4];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const bool row = ch < cb && k0 + e < n;
    const uint16_t* s = p + (row ? (long)(k0 + e) * 4 * n : 0);
    if (n % 8 == 0) {
      const uint4 v = *(const uint4*)(s + (u0 < n ? u0 : 0));
      const bool in = row && u0 < n;
      r[e][0] = in ? v.x : 0u; r[e][1] = in ? v.y : 0u; r[e][2] = in ? v.z : 0u; r[e][3] = in ? v.w : 0u;
    } else {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const unsigned x = row && u0 + 2 * h < n ? s[u0 + 2 * h] : 0u, y = row && u0 + 2 * h + 1 < n ? s[u0 + 2 * h + 1] : 0u;
        r[e][h] = x | (y << 16);
      }
    }
  }
  const auto scaled = [](unsigned lo16, unsigned hi16) {
    return (__float_as_uint(__uint_as_float(lo16 << 16) * kScale) >> 16) | (__float_as_uint(__uint_as_float(hi16 << 16) * kScale) & 0xffff0000u);
  };
  uint4* o = out + (((((long)j * I + i) * 4 + gate) * 2 + ((u8 >> 1) & 1)) * 16 + ch) * 64 + (kk & 3) * 16 + (u8 & 1) * 8;
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    unsigned v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = h & 1 ? r[e][h >> 1] >> 16 : r[e][h >> 1] & 0xffffu;
    o[h] = make_uint4(scaled(v[0], v[1]), scaled(v[2], v[3]), scaled(v[4], v[5]), scaled(v[6], v[7]));
  }
}

int ranges_for(int n) { return cdiv(n, 512); }             // K ranges of the forward kernel
int fwd_grid(int n) { return 8 * cdiv(cdiv(n, 32), 8) * ranges_for(n); }
int bwd_grid(int n) { return 16 * cdiv(n, kBlk); }

// Clear before a launch: the rings, and the words in which columns find out that they share an XCD.
template <typename A>
ZeroRegions regions_of(const A& a, bool first) {
  ZeroRegions z;
  z.add(a.ring, a.ring_bytes);
  z.add(a.xcc, 256 * 4);
  if (first) z.add(a.sync, 4);                             // (a wait that expired in an earlier direction stays on record)
  return z;
}
template <typename K, typename A>
hipError_t launch_blocks(K one, K two, int blocks, A a, bool cleared, hipStream_t s) {
  for (int row0 = 0; row0 < a.B; row0 += kSlab) {          // (rows never interact; a launch walks all steps of its rows)
    a.row0 = row0;
    hipError_t e;
    if ((row0 > 0 || !cleared) && (e = launch_fill_zero_many(regions_of(a, row0 == 0 && a.first), s)) != hipSuccess) return hipErrorLaunchFailure;
    void* args[] = {&a};
    const void* kernel = (const void*)(a.B - row0 <= 16 ? one : two);
    e = a.plain_launch ? hipLaunchKernel(kernel, dim3(blocks), dim3(256), args, 0, s) : hipLaunchCooperativeKernel(kernel, dim3(blocks), dim3(256), args, 0, s);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return row0 == 0 ? hipErrorCooperativeLaunchTooLarge : hipErrorLaunchFailure;
    }
  }
  return hipSuccess;
}

}  // namespace

// Widths whose W_h does not fit persistent.hip's split and fits this one; all work-groups (256 at most) must be resident together.
bool loop_block_width(int n) { return n > 1024 && n <= 2048; }
bool loop_block_fits(int B, int n, long ld_out) {
  const long lim = kParked;                                // offsets inside a frame are 32 bits
  return loop_block_width(n) && (long)B * 16 * n < lim && (long)B * ld_out * 2 < lim && std::min(device_capacity((const void*)block_fwd_kernel<1>), device_capacity((const void*)block_fwd_kernel<2>)) >= fwd_grid(n) &&
         std::min(device_capacity((const void*)block_bwd_kernel<1>), device_capacity((const void*)block_bwd_kernel<2>)) >= bwd_grid(n);
}
// A launch is 32 rows of one direction and walks all steps, while the per-step kernels take every row and both directions in one pass over
// W_h: with many rows, above all of the narrower layers, those are faster (n = 1032, 256 rows, both directions, us a step: 82 forward and 104
// backward here, 32 and 38 there; n = 2048, 64 rows, one direction: 9.4 and 10.1 here, 14.8 and 23.5 there).  Both sides as they were measured,
// in us, for n from 1032 to 2048, 4 to 256 rows, 2 to 100 steps, one and two directions, plain and cooperative launches (624 shapes, each
// pass both ways: the choice is within 5 % of the faster side in 98 % of them, never 1.35 times it, while always one launch was up to 6.4
// times the other).  A column's tasks are two to a member up to 1536 units forward and 1920 backward, one above.
bool loop_block_pays(int T, int B, int n, int ndir, bool plain_launch, bool backward) {
  const double w = (double)n * n / (2048.0 * 2048.0), nr = (double)n * ndir * B * 1e-5;
  const int slabs = cdiv(B, kSlab), half = B % kSlab != 0 && B % kSlab <= 16, whole = slabs - half;      // half: a slab of one row tile
  const double start = 14.5 + (plain_launch ? 0.0 : 18.2);
  double here, there;
  if (backward) {
    const bool one_task = n > 1920;
    here = 24 + ndir * (23 * w + slabs * start + T * (whole * (one_task ? 5.45 : 6.85) + half * (one_task ? 4.3 : 3.8)));
    there = 42 + ndir * 51 * w + T * std::max(2 + 9.6e-3 * n + 3.8 * nr, 10.2 * nr);
  } else {
    const bool one_task = n > 1536;
    here = 10.5 + ndir * (17.8 * w + slabs * start + T * (whole * (one_task ? 4.05 : 4.65) + half * (one_task ? 3.4 : 3.15)));
    there = 23.5 + ndir * 20.5 * w + T * std::max(2.2 + 3.1e-3 * n + 5.45 * nr + 2.1 * (ndir - 1) * w, 6.9 * nr);
  }
  return here < there;
}
size_t loop_block_ring_bytes(int n) { return 2 * (64 * 2048 + (size_t)cdiv(n, 32) * 4 * 4 * 4096); }
size_t loop_block_ring_bytes_bwd(int n) {
  const size_t nb = cdiv(n, kBlk);
  return 2 * (nb * 32768 + nb * nb * 16 * 1024) + 16384;   // (what unpredicated loads read behind the last share)
}
size_t loop_block_wh_bytes(int n) { return (size_t)cdiv(n, 32) * ranges_for(n) * 8 * 16 * 1024; }
hipError_t launch_pack_blocks(const void* W_h, const BlockFwdArgs& a, hipStream_t s) {
  const ZeroRegions z = regions_of(a, a.first);
  if (z.overflow) return hipErrorInvalidValue;
  const int columns = ranges_for(a.n) * 8, packs = cdiv(a.n, 64);
  hipLaunchKernelGGL(pack_blocks_kernel, dim3(columns, packs + cdiv(z.first_block[z.count], columns)), dim3(256), 0, s, (const bf16_t*)W_h, (uint4*)a.W, a.n, ranges_for(a.n), z, packs);
  return hipGetLastError();
}
hipError_t launch_block_fwd(const BlockFwdArgs& a, hipStream_t s) {
  BlockFwdArgs c = a;
  c.ni = ranges_for(a.n);
  return launch_blocks(block_fwd_kernel<1>, block_fwd_kernel<2>, fwd_grid(a.n), c, true, s);
}
hipError_t launch_block_bwd(const BlockBwdArgs& a, hipStream_t s) { return launch_blocks(block_bwd_kernel<1>, block_bwd_kernel<2>, bwd_grid(a.n), a, false, s); }

}  // namespace lstm
