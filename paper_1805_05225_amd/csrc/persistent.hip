// Single-launch recurrent kernels: the whole time loop of a layer in ONE launch (bfloat16 storage).
//
// The per-step kernels pay a launch per time step and re-read their W_h slice from the memory
// system every step.  Here each work-group (32 hidden units x 8 batch rows, or x 16 rows for batches
// that the 8-row form cannot hold in one launch) loads its slice of the packed W_h into registers once and
// then walks all T steps.
//
// Only h_t (forward) or partial sums of Dh (backward) cross work-groups.  Measurements on this device
// showed that a counter barrier is the wrong tool: atomics on one address serialise at ~16 ns each
// (4 us for 256 work-groups) and agent-scope fences cost microseconds more.  So there is no
// barrier and no fence here.  The exchanged data lives in a two-slot ring whose every 8-byte unit
// holds its values AND a tag of the step that wrote it (four bf16 values, the tag one bit that their
// range leaves free), written with one 64-bit store and read with cache-bypassing 16-byte loads.  A consumer simply re-reads an operand until
// its tags show the step it is waiting for: value and "ready" flag arrive in the same atomic
// unit, so no ordering between different addresses is ever needed.
//
// Two ring slots suffice: a work-group writes slot s for step t+1 only after it has seen every
// tag of step t, i.e. after every work-group has finished step t and therefore finished reading
// slot s (which held step t-1).
//
// Every wait is bounded: after `spin_limit` polls the wave raises the error word sync[0], stops
// waiting for the rest of the launch and runs to the end (results are then invalid and the word
// says so); every other wave notices the word in its own wait loop and does the same, so the
// grid always drains.  The grid is checked against what the device holds at once; the launch is
// cooperative unless the caller vouches that nothing else occupies the device.
#include "exchange_dev.h"
#include <type_traits>
#include <algorithm>
#include <map>
#include <mutex>

namespace lstm {
namespace {


// Optional in-kernel phase clocks (build with -DLSTM_PROF; prints from a few work-groups at the end).
#ifdef LSTM_PROF
#define PROF_DECL long long pt_[8] = {0, 0, 0, 0, 0, 0, 0, 0}; long long pc_ = wall_clock64(); unsigned npoll_ = 0, nredo_ = 0;
#define PROF_MARK(i) { long long now_ = wall_clock64(); pt_[i] += now_ - pc_; pc_ = now_; }
#define PROF_POLLS(n) npoll_ += (n);
#define PROF_REDO(n) nredo_ += (n);
#define PROF_DUMP(name, steps) if ((tid & 63) == 0 && (blockIdx.x % 23) == 0 && blockIdx.y == 0) \
  printf("%s wg(%d,%d,%d) wave %d: ns/step sample %lld stream %lld mma %lld red+cell %lld publish %lld other %lld polls/step %.2f loads fetched again per 1000 steps %.1f\n", name, blockIdx.x, blockIdx.y, blockIdx.z, (int)(threadIdx.x >> 6), \
         pt_[5] * 10 / (steps), pt_[0] * 10 / (steps), pt_[1] * 10 / (steps), pt_[2] * 10 / (steps), pt_[3] * 10 / (steps), pt_[4] * 10 / (steps), (double)npoll_ / (steps), 1000.0 * nredo_ / (steps));
#else
#define PROF_DECL
#define PROF_MARK(i)
#define PROF_POLLS(n)
#define PROF_REDO(n)
#define PROF_DUMP(name, steps)
#endif
// Ring reads.  One wavefront owns chunks kc = wave + 4*it of its row tile.  Reads of freshly written
// remote data are latency-bound per compute unit and degrade when more than ~12 KiB per wavefront is in
// flight, so (a) a wave first polls the first two of its loads until they show the awaited tag, which is cheap
// while the producers are still busy, and only then (b) fetches the rest, checking every tag; a load whose tags
// are stale is fetched again on its own (fix_up_batch, or an immediate re-issue through LDS), never the whole set.
//
// Nothing in the stream is predicated.  The buffer descriptor covers exactly the nkc chunks of the row tile,
// so a load past the end (chunks the template bound adds beyond nkc, lanes whose rows this work-group does
// not own: their offset is parked far outside) returns zeros from the bounds check without touching memory.
// Padding units inside the ring hold zero values (nobody writes them after the initial fill), so masking off
// the tags is all the clean-up an operand needs.  Keeping branches and lane masks out of this loop
// matters: with them the instruction stream between two loads, not the memory system, set the step time.
// Order in which a work-group walks the nitv loads of its row tile: rotated by `rot`, so that the work-groups of
// one XCD, which all read the same tile at the same time, do not all ask the same L2 channel for the same lines.
__device__ __forceinline__ int rot_index(int i, int rot, int nitv) {
  const int j = i + rot;
  return i >= nitv ? i : (j >= nitv ? j - nitv : j);
}
template <typename Reader> struct RingReads {           // what readers have in common; where a load lies is the reader's
  __amdgpu_buffer_rsrc_t rs;
  unsigned tag;                          // the awaited tag as it sits in the upper half of a unit's second dword
  unsigned* err;
  unsigned limit;

  __device__ __forceinline__ int it_of(int i) const { return static_cast<const Reader*>(this)->it_of(i); }
  __device__ __forceinline__ u32x4 load_it(int it) const {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, static_cast<const Reader*>(this)->offset(it), 0, kSc1);
  }
  __device__ __forceinline__ bool expects(int it) const { return static_cast<const Reader*>(this)->expects(it); }   // does this lane's unit of load `it` carry a tag?
  // Tag differences of one load, per lane: a bit above the low half iff one of the lane's two tags is not `tagw >> 16`.
  // Lanes whose units carry no tag (padding inside the ring, chunks past the end) report nothing, whatever they read.
  __device__ __forceinline__ unsigned tag_diff(const u32x4& x, int it, unsigned tagw) const {
    const unsigned t = (x[1] ^ tagw) | (x[3] ^ tagw);
    return expects(it) ? t & kLLFwdTagBit : 0u;
  }
  __device__ __forceinline__ unsigned stale_bits(const u32x4& x, int it) const {
    const unsigned d = ((x[1] >> 16) ^ tag) | ((x[3] >> 16) ^ tag);
    return expects(it) ? d & (kLLFwdTagBit >> 16) : 0u;
  }
  // The poll after its first, mostly successful, look (which stays in line: a loop around it costs its branches in every step).
  template <typename L, typename S>
  __device__ __forceinline__ void poll_again(bool& dead, L&& loads, S&& stale) const {
    for (unsigned poll = 1;; ++poll) {
      loads();
      if (!stale()) return;
      if (poll >= limit || ((poll & 63u) == 63u && ld_relaxed(err) != 0u)) {
        st_relaxed(err, 1u);
        dead = true;
        return;
      }
    }
  }
  // Second pass over the loads marked in `redo`, all of them in flight at once: every round fetches those still
  // marked, hands the ones whose tags have all turned to `use` (operand as loaded, tags included) and keeps the
  // rest for the next round (bounded).
  template <int NIT, int OFF = 0, typename F>
  __device__ __forceinline__ void fix_up_batch(unsigned long long redo, bool& dead, F&& use) const {
    redo &= ((1ull << NIT) - 1ull) << OFF;                    // loads OFF .. OFF + NIT - 1 of the stream
    for (unsigned poll = 0; redo != 0ull && !dead; ++poll) {
      u32x4 x[NIT];
#pragma unroll
      for (int i = 0; i < NIT; ++i)
        if ((redo >> (i + OFF)) & 1ull) x[i] = load_it(it_of(i + OFF));
#pragma unroll
      for (int i = 0; i < NIT; ++i) {
        if (!((redo >> (i + OFF)) & 1ull)) continue;
        if (__builtin_amdgcn_ballot_w64(stale_bits(x[i], it_of(i + OFF)) != 0u) == 0ull) {
          use(i + OFF, x[i]);
          redo &= ~(1ull << (i + OFF));
        }
      }
      if (redo != 0ull && (poll >= limit || ((poll & 63u) == 63u && ld_relaxed(err) != 0u))) {
        st_relaxed(err, 1u);
        dead = true;
      }
    }
  }
};
struct RingReader : RingReads<RingReader> {
  int rot, nitv;                         // load i of the stream fetches iteration (i + rot) mod nitv of the row tile
  unsigned voff;                         // byte offset of this lane's first load (parked out of range if the lane is off)
  unsigned it_bytes;                     // byte distance between consecutive loads of a lane
  int lim, lim_step;                     // load `it` carries awaited tags for this lane iff lim_step*it < lim
  __device__ __forceinline__ int it_of(int i) const { return rot_index(i, rot, nitv); }
  __device__ __forceinline__ unsigned offset(int it) const { return voff + (unsigned)it * it_bytes; }
  __device__ __forceinline__ bool expects(int it) const { return lim_step * it < lim; }
};

// `nchunk_valid` counts the 16-lane groups (quarter chunks) that producers write; `lane_on` is false for lanes
// whose fragment rows belong to another work-group.
__device__ __forceinline__ RingReader make_reader(const uint4* base, int nkc, int nchunk_valid, int wave, int lane, unsigned tag,
                                                   unsigned* err, unsigned limit, int rot, bool lane_on = true) {
  RingReader r;
  r.nitv = (nkc + 3) / 4; r.rot = rot;
  r.rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, nkc * 1024, kBufFlags);
  r.voff = lane_on ? (unsigned)(wave * 1024 + lane * 16) : 0x7ff00000u;
  r.it_bytes = 4096u;
  r.lim = lane_on ? nchunk_valid - (lane >> 4) - 4 * wave : -0x40000000;
  r.lim_step = 16;
  r.tag = tag; r.err = err; r.limit = limit;
  return r;
}

// Reader for a work-group that owns only 8 of a row tile's 16 rows (`half` selects which).  A load would
// leave half the lanes idle, and the time of a ring read goes with the number of loads, not their bytes; so one
// load serves TWO chunks: lanes whose fragment row is below 8 fetch our rows of chunk wave + 8*it, the others
// our rows of chunk wave + 8*it + 4; rows_from_low and rows_from_high make the two operands of it.
__device__ __forceinline__ RingReader make_reader_half(const uint4* base, int nkc, int nchunk_valid, int wave, int lane, int half,
                                                        unsigned tag, unsigned* err, unsigned limit, int rot) {
  RingReader r;
  r.nitv = (nkc + 7) / 8; r.rot = rot;
  const int row = lane & 15, g = lane >> 4, second = row >> 3;
  r.rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, nkc * 1024, kBufFlags);
  r.voff = (unsigned)((wave + 4 * second) * 1024 + (g * 16 + half * 8 + (row & 7)) * 16);
  r.it_bytes = 8192u;
  r.lim = nchunk_valid - g - 4 * wave - 16 * second;
  r.lim_step = 32;
  r.tag = tag; r.err = err; r.limit = limit;
  return r;
}
// The same with the chunks in the order of the 16-row kernel (load i: its chunks 2i and 2i + 1), so that sums come out as they do there: a
// batch may take either, and results that differ in the last place pick other frames in a maximum over time further up.
template <int NL> struct PairReader : RingReads<PairReader<NL>> {
  unsigned off[NL]; int lim[NL];
  __device__ __forceinline__ int it_of(int i) const { return i; }
  __device__ __forceinline__ unsigned offset(int i) const { return off[i]; }
  __device__ __forceinline__ bool expects(int i) const { return lim[i] > 0; }
};
template <int NL>
__device__ __forceinline__ PairReader<NL> make_reader_pairs(const uint4* base, int nkc, int nchunk_valid, int wave, int lane, int half,
                                                            unsigned tag, unsigned* err, unsigned limit, int rot) {
  PairReader<NL> r;
  const int row = lane & 15, g = lane >> 4, second = row >> 3;
  r.rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, nkc * 1024, kBufFlags);
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int kc = wave + 4 * rot_index(2 * i + second, rot, (nkc + 3) / 4);
    r.off[i] = (unsigned)(kc * 1024 + (g * 16 + half * 8 + (row & 7)) * 16);
    r.lim[i] = nchunk_valid - g - 4 * kc;
  }
  r.tag = tag; r.err = err; r.limit = limit;
  return r;
}
// two floats -> two bf16 (round to nearest even) in one register, low half first
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_;
  const bf16x2_ r = __builtin_convertvector((f32x2_){lo, hi}, bf16x2_);
  return __builtin_bit_cast(unsigned, r);
}
// Streaming stores of the recurrent kernels (every byte touched once): marked non-temporal so that they do not
// push the exchange ring, which is re-read every step, out of the L2.
__device__ __forceinline__ void st_stream(unsigned short* p, unsigned short v) { __builtin_nontemporal_store(v, p); }

// --- W_h in accumulation registers ---------------------------------------------------------------------------
// The register file of a wavefront is 256 architectural + 256 accumulation registers.  A W_h slice larger than
// what is left of the first 256 is parked by the compiler in accumulation registers and copied back, four moves
// per MFMA, before every use - with one wavefront per SIMD those moves are on the critical path.  MFMA can read
// its B operand from accumulation registers directly, so the slice is loaded straight into them and the products
// are issued through inline assembly.  The compiler does not see an MFMA in that text, so the wait states the
// hardware needs between the last MFMA and the first read of its result are inserted by hand (mfma_settle).
__device__ __forceinline__ u32x4 load_to_agpr(const uint4* p) {
  u32x4 r;
  asm volatile("global_load_dwordx4 %0, %1, off" : "=a"(r) : "v"(p) : "memory");
  return r;
}
__device__ __forceinline__ void agpr_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// acc += A (16 rows x 32 k, vector registers) x B (32 k x 16 columns, accumulation registers)
__device__ __forceinline__ void mfma_b_agpr(f32x4& acc, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_b_vgpr(f32x4& acc, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// --- eight rows, no wasted half --------------------------------------------------------------------------------
// The dense 16x16x32 product of a work-group of 8 rows multiplies 8 rows of nothing.  The sparse instruction (16x16x64, the same 16
// cycles) takes an A of which two of every four k are stored, and WHICH two may differ from row to row.  Fragment rows 0-7 and 8-15
// both hold our rows; the former say that their values belong to the k that are 0 or 1 mod 4, the latter 2 or 3 mod 4 (kSparseLow,
// kSparseHigh: the positions, two bits each).  With the weights of one column tile at the former k of B and those of the next tile at the
// latter, one instruction does the work of two: fragment rows 0-7 of the result are the first tile's, rows 8-15 the second's.  The bits
// are those of the dense product (51200 sums of 8 x 32 products compared on the device).
// Lane l supplies for A row l%16 the eight stored values of k = 16 (l/16) .. +15, for B column l%16 the k 8 (l/16) .. +7 in the
// first four registers and 32 + those in the last four (measured on the device).
constexpr int kSparseLow = 0x44444444, kSparseHigh = (int)0xeeeeeeeeu;
// What element e of lane group g holds in B register set `set` (0, 1): column tile, and which of the 32 k.
__host__ __device__ constexpr int sparse_tile(int e) { return (e >> 1) & 1; }
__host__ __device__ constexpr int sparse_k(int set, int g, int e) { return 8 * (2 * set + (g >> 1)) + ((g & 1) * 2 + (e >> 2)) * 2 + (e & 1); }
typedef __attribute__((ext_vector_type(8))) unsigned u32x8;
// two register sets as one operand (behind agpr_loads_done: until then nothing may copy them)
__device__ __forceinline__ u32x8 agpr_join(u32x4& lo, u32x4& hi) {
  asm volatile("" : "+a"(lo), "+a"(hi));
  u32x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  asm volatile("" : "+a"(r));            // (an accumulation-register value from here on: no copy at its uses)
  return r;
}
__device__ __forceinline__ void smfmac_b_agpr(f32x4& acc, const u32x4& a, const u32x8& b, int idx) {
  asm volatile("v_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3" : "+v"(acc) : "v"(a), "a"(b), "v"(idx));
}
// The operands of a load whose lanes hold one chunk in fragment rows 0-7 and another in rows 8-15 (make_reader_half): its first
// (second) chunk in all rows.  Rotated by 8 inside each row of 16 lanes, written to the upper (lower) eight only.
__device__ __forceinline__ unsigned rows_from_low(unsigned v) { return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xf, 0xc, false); }
__device__ __forceinline__ unsigned rows_from_high(unsigned v) { return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xf, 0x3, false); }
// acc = A x B: the first product of a chain takes the constant 0 as its addend, so the accumulators need no clearing
// (64 moves per step in the backward kernel, and the wait states between them and the first MFMA).  The result may not share
// registers with an operand: early clobber.
__device__ __forceinline__ void mfma_b_agpr_first(f32x4& acc, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "a"(b));
}
// The float MFMA (16x16x4): one float of A and one of B per lane.
__device__ __forceinline__ void mfma4_b_vgpr(f32x4& acc, float a, float b) {
  asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_settle(f32x4& a0) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(a0)); }
// Wait states between the last ordinary (vector ALU, DPP, LDS) write of registers and an MFMA reading them.  For
// MFMAs it emits itself the compiler knows what the hardware needs; for these it cannot, and an MFMA issued right
// behind DPP moves was observed to read the old register contents.
#ifndef LSTM_OPERAND_NOPS
#define LSTM_OPERAND_NOPS "7"
#endif
// s_waitcnt vmcnt(n) for an n that is constant after unrolling (0 .. 15; the instruction takes an immediate).
// Where a kernel consumes a ring load while younger stores are in flight it waits with this, n = the number of
// YOUNGER LOADS: loads return in the order of issue among themselves, but stores were seen to be acknowledged ahead of
// older loads that bypass L2, so a count that includes the younger stores - what the compiler emits - can be reached
// while the load is still on its way.
// The wait names the registers it is for: an assembly statement that "rewrites" them, so that no instruction reading them can
// be scheduled in front of it (in straight-line code the compiler would otherwise be free to, with only its own wait before them).
#define LSTM_WAIT_CASE(N) case N: asm volatile("s_waitcnt vmcnt(" #N ")" : "+v"(x)); break;
__device__ __forceinline__ void wait_loads_but(int n, u32x4& x) {
  switch (n < 15 ? n : 15) {
    LSTM_WAIT_CASE(0) LSTM_WAIT_CASE(1) LSTM_WAIT_CASE(2) LSTM_WAIT_CASE(3) LSTM_WAIT_CASE(4) LSTM_WAIT_CASE(5) LSTM_WAIT_CASE(6) LSTM_WAIT_CASE(7)
    LSTM_WAIT_CASE(8) LSTM_WAIT_CASE(9) LSTM_WAIT_CASE(10) LSTM_WAIT_CASE(11) LSTM_WAIT_CASE(12) LSTM_WAIT_CASE(13) LSTM_WAIT_CASE(14)
    default: asm volatile("s_waitcnt vmcnt(15)" : "+v"(x)); break;
  }
}
#undef LSTM_WAIT_CASE
// f(integral_constant<0>) ... f(integral_constant<N - 1>): a loop whose counter is a constant expression in the body
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}
__device__ __forceinline__ void operands_settle(u32x4& a) { asm volatile("s_nop " LSTM_OPERAND_NOPS : "+v"(a)); }
__device__ __forceinline__ void operands_settle(u32x4& a, u32x4& b) { asm volatile("s_nop " LSTM_OPERAND_NOPS : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void operands_settle(u32x4& a, u32x4& b, u32x4& c, u32x4& d) {
  asm volatile("s_nop " LSTM_OPERAND_NOPS : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
__device__ __forceinline__ void operands_settle(f32x4& a, f32x4& b, f32x4& c, f32x4& d) {
  asm volatile("s_nop " LSTM_OPERAND_NOPS : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
// 20 wait states: more than any MFMA of this shape needs before its result may be read or overwritten
__device__ __forceinline__ void mfma_settle(f32x4& a0, f32x4& a1) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(a0), "+v"(a1)); }
__device__ __forceinline__ void mfma_settle(f32x4& a0, f32x4& a1, f32x4& a2, f32x4& a3) {
  asm volatile("s_nop 15\n\ts_nop 3" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3));
}
__device__ __forceinline__ void mfma_settle(f32x4& a0, f32x4& a1, f32x4& a2, f32x4& a3, f32x4& a4, f32x4& a5, f32x4& a6, f32x4& a7) {
  asm volatile("s_nop 15\n\ts_nop 3" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(a4), "+v"(a5), "+v"(a6), "+v"(a7));
}

// Work-group -> (unit tile, row group, direction).  Work-groups are dealt to the 8 XCDs round-robin in launch order, and
// the work-groups of one (direction, row group) exchange data every step.  map.gpx > 0: XCD x runs the groups x, x + 8, ...
// (gpx of them at most; the grid is sized for 8 gpx groups and the surplus leaves at once), so that every exchange stays inside one
// XCD - also with fewer groups than XCDs, where spreading a group over two of them to use them all made a step 2.7 us instead
// of 1.6 (one sentence, both directions, n = 1000).  gpx = 0 (more work-groups per XCD than it has compute units): where the shape
// allows it each XCD serves a single group.  Any bijection is correct; these are only faster.
struct WgCoord { int tile, rt, dir, base; bool live; };      // base: place of the group's first word in the XCD table
__device__ __forceinline__ WgCoord wg_coord(const GridMap& m, int ndir) {
  const int groups = m.nrow * ndir, total = m.ntile * groups, lin = blockIdx.x;
  int tile = lin % m.ntile, group = lin / m.ntile;
  if (m.gpx > 0) {
    const int slot = lin >> 3;
    group = (lin & 7) + 8 * (slot / m.ntile);
    tile = slot % m.ntile;
  } else if (groups <= 8 && 8 % groups == 0 && total % 8 == 0) {
    const int xcd = lin & 7, slot = lin >> 3, per_group = 8 / groups;     // XCDs per group
    group = xcd % groups;
    tile = xcd / groups + per_group * slot;
  }
  // (told to be wave-uniform: divisions leave them in vector registers, and a buffer descriptor formed from those is applied
  // lane by lane in a loop)
  tile = __builtin_amdgcn_readfirstlane(tile);
  group = __builtin_amdgcn_readfirstlane(group);
  const int dir = __builtin_amdgcn_readfirstlane(group / m.nrow);
  WgCoord c = {tile, group - dir * m.nrow, dir, group * m.ntile, group < groups && tile < m.ntile};     // (a grid may be meant for more groups)
  return c;
}

// --- rows one behind the other -----------------------------------------------------------------------------------
// More rows than a launch of the 8-row kernels holds, of different lengths: the launch's row places (`slots`, eight to a group) take rows
// one after the other, so that a layer takes about (all frames / slots) steps instead of the longest row's for every 16 rows.  What a
// place does in a step is a word of a table that the set-up launch writes from the lengths (pack_rows_body): frame t * B + b, and
// whether it is a row's first or last.  Nothing crosses from row to row: a row's last step publishes zeros, its first takes the
// caller's state, and h0 W_h is in its pre-activations already (see `started`).
// 64 rows of 20-80 frames, n = 1000, both directions: 80 steps of 2.5 us on the 16-row kernels, 100 of 1.45 (backward 1.65) here: a layer 204 -> 162 us and 203 -> 172.
constexpr unsigned kRowValid = 1u << 28, kRowFirst = 1u << 29, kRowLast = 1u << 30, kRowFrame = kRowValid - 1u;
constexpr int kTabSteps = 512;                             // steps whose table words are kept in LDS (and a few more, asked for ahead)
// A uniform value, held where buffer descriptors are formed from it.
__device__ __forceinline__ unsigned in_sgpr(unsigned v) {
  v = __builtin_amdgcn_readfirstlane(v);
  asm("" : "+s"(v));
  return v;
}
// A load on a path that few steps take, waited for there: the compiler would wait where the paths meet, for everything in flight.
__device__ __forceinline__ float rare_load(const float* p) {
  float v = *p;
  asm volatile("" : "+v"(v));
  return v;
}
// byte offset of a word's frame (frames and their sizes are below 2^24)
__device__ __forceinline__ unsigned frame_off(unsigned e, unsigned bytes) { return __umul24(e & kRowFrame & 0xffffffu, bytes); }
template <bool PACKED> struct RowTable {
  static constexpr int kSteps = PACKED ? kTabSteps + 8 : 1;
  unsigned (*lds)[8]; const unsigned* mem; int steps, slot;
  // words of the steps from s0 on (s0 a multiple of kTabSteps); all threads of the work-group
  __device__ __forceinline__ void load(int s0) const {
    if constexpr (PACKED) {
      __syncthreads();
      for (int i = threadIdx.x; i < kSteps * 8; i += 256) lds[i >> 3][i & 7] = s0 + (i >> 3) < steps ? mem[(long)s0 * 8 + i] : 0u;
      __syncthreads();
    }
  }
  __device__ __forceinline__ unsigned at(int step, int now) const { return PACKED ? lds[step - (now & ~(kTabSteps - 1))][slot] : 0u; }
};

// --- W_h as it lies in memory ------------------------------------------------------------------------------------
// A fragment has a column's k side by side, W_h a row's units: 16 k x 32 units of a gate are one load that goes straight into LDS (64 bytes a row), and
// ds_read_b64_tr_b16 turns them on the way out (sixteen lanes name eight bytes each of four rows of sixteen units and get a unit each).  Saves the packed
// copy (n = 1000, both directions: 16 MB read, 17 MB written, 12 us).  A loop's start is then 1.5 us longer if W_h is in the last-level
// cache and 5 if not, so this is for layers whose set-up fetches it there beforehand (prep_zx_kernel).  Neighbouring work-groups ask for neighbouring pieces at
// the same time: with the chunks rotated tile by tile, as for packed weights, a start took 4 us more.
// A chunk of 32 k is 8 KiB of a wavefront's buffer, kWChunks of them in flight.  n is a multiple of 8; units and rows from n on are outside the descriptor: zeros.
constexpr int kWChunks = 3;
typedef __attribute__((ext_vector_type(4))) short s16x4;
__device__ __forceinline__ u32x2 turned(const char* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}
// chunk_of(it): the chunk of the wavefront's it-th operands; use(it, rows): they are at `rows`, [gate][k][64 bytes].
template <int ITS, typename C, typename U>
__device__ __forceinline__ void walk_w_rows(const void* W, int n, int tile2, char (&buf)[kWChunks][8192], int lane, C&& chunk_of, U&& use) {
  static_assert(kWChunks == 3, "the counted waits below");
  const unsigned ldw = 8u * n, u0 = tile2 * 32 + (lane & 3) * 8;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, n * ldw, kBufFlags);
  const unsigned off0 = u0 < (unsigned)n ? (lane >> 2) * ldw + u0 * 2u : 0x7ff00000u;
  const unsigned to = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&buf[0][0]);
  auto ask = [&](int it) __attribute__((always_inline)) {
    const unsigned row0 = chunk_of(it) * 32;
#pragma unroll
    for (int i = 0; i < 8; ++i)                            // gate i / 2, rows 16 (i & 1) .. + 15
      asm volatile("s_add_u32 m0, %0, %1\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds" ::"s"(to), "i"((it % kWChunks) * 8192 + i * 1024),
                   "v"(off0 + ((row0 + (i & 1) * 16u) * ldw + (i >> 1) * 2u * n)), "s"(rs) : "memory", "scc");
  };
#pragma unroll
  for (int it = 0; it < (ITS < kWChunks ? ITS : kWChunks); ++it) ask(it);
#pragma unroll
  for (int it = 0; it < ITS; ++it) {                       // (loads complete in the order of issue)
    if (it + 2 < ITS) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if (it + 1 < ITS) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    use(it, buf[it % kWChunks]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // (read out, before it is written again)
    if (it + kWChunks < ITS) ask(it + kWChunks);
  }
}

// ------------------------------------------------------------------------------------------------
// forward: z[8 rows, 4 gates x 32 units] = h[8 rows, K] W[K, 128].  A work-group owns 32 units for 8 batch rows
// (half a row tile); one load serves two chunks (see make_reader_half), one product two column tiles (see smfmac_b_agpr).  The W_h
// slice fills the 256 accumulation registers of every lane (n = 1024).
template <bool PACKED> struct Fwd8Steps {
  static constexpr int kAhead = 2;                       // frames of x W_x + b that are fetched together (fetch_zx below)
  alignas(16) float red[2][4][8][129];                   // two copies, used by even and odd steps: one barrier per step
  alignas(16) float zxs[kAhead][4][2][4][32];            // [frame][wavefront][row][gate][unit]: a wavefront reads back what it asked for
  alignas(16) unsigned tab[RowTable<PACKED>::kSteps][8];
};
// (first the rows of W_h, [wavefront][chunk in flight], where they come as they lie in memory)
template <bool PACKED, bool ROWS> union Fwd8Lds { Fwd8Steps<PACKED> step; char w[4][ROWS ? kWChunks : 1][ROWS ? 8192 : 16]; };
template <int NL, bool PACKED, bool ROWS = false>          // ring loads per wavefront and step: n <= 256 NL; rows one behind the other; W_h as it lies in memory
__device__ __forceinline__ void fwd8_body(const PFwdArgs& a, Fwd8Lds<PACKED, ROWS>& lds_) {
  auto& lds = lds_.step;
  constexpr int kAhead = Fwd8Steps<PACKED>::kAhead;
  auto& red = lds.red;
  auto& zxs = lds.zxs;
  auto& tab_lds = lds.tab;
  const WgCoord wg = wg_coord(a.map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const PFwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int tile2 = wg.tile, rt = a.rt0 + (wg.rt >> 1), half = wg.rt & 1;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nkc = a.nkc, n = a.n, B = a.B, T = a.T;
  const int ntiles16 = (n + 15) / 16;
  unsigned* err = a.sync;
  bool dead = false;

  const int nitv = PACKED ? (nkc + 3) / 4 : (nkc + 7) / 8, rot = ROWS ? tile2 * nitv / ((n + 31) / 32) : tile2 % nitv;
  // Operands 2p, 2p + 1 of a gate are the two chunks that load p of the stream fetches.  Those of chunks past the end are loaded
  // from a chunk of zeros that the host keeps behind the packed weights.
  u32x4 w4[2 * NL][4][2];
  if constexpr (ROWS) {
    // rows k, k + 1 of the first column tile, then of the second: what elements 0 - 3 of lane group g hold (4 - 7: k + 2, k + 3)
    const int at = ((lane >> 4) * 4 + ((lane >> 2) & 1)) * 64 + ((lane >> 3) & 1) * 32 + (lane & 3) * 8;
    walk_w_rows<2 * NL>(d.Wf, n, tile2, lds_.w[wave], lane, [&](int it) { return wave + 4 * (2 * rot_index(it >> 1, rot, nitv) + (it & 1)); },
        [&](int it, const char* rows) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int set = 0; set < 2; ++set) {
              const u32x2 lo = turned(rows + q * 2048 + set * 1024 + at), hi = turned(rows + q * 2048 + set * 1024 + 128 + at);
              w4[it][q][set] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
            }
        });
    __syncthreads();                                       // (the buffer is the steps' from here on)
  } else {
#pragma unroll
  for (int it = 0; it < 2 * NL; ++it) {
    const int kc = wave + 4 * (PACKED ? rot_index(it, rot, nitv) : 2 * rot_index(it >> 1, rot, nitv) + (it & 1));
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int set = 0; set < 2; ++set)
        w4[it][q][set] = load_to_agpr(kc < nkc ? &d.Wf[(((long)(tile2 * 4 + q) * nkc + kc) * 2 + set) * 64 + lane] : &d.Wzero[lane]);
  }
  agpr_loads_done();
  }
  u32x8 w[2 * NL][4];
#pragma unroll
  for (int it = 0; it < 2 * NL; ++it)
#pragma unroll
    for (int q = 0; q < 4; ++q) w[it][q] = agpr_join(w4[it][q][0], w4[it][q][1]);
  const int sparse = (lane & 8) ? kSparseHigh : kSparseLow;

  const int r8 = tid >> 5, u = tid & 31;                 // pointwise pair of this thread: row r8 of the half, unit u of 32
  const int b = PACKED ? 0 : rt * 16 + half * 8 + r8, j = tile2 * 32 + u;
  const bool active = b < B && j < n;
  const RowTable<PACKED> tab = {tab_lds, PACKED ? d.tab + (long)wg.rt * a.tab_steps * 8 : nullptr, PACKED ? __builtin_amdgcn_readfirstlane(a.steps[wg.rt]) : T, r8};
  float c = 0.f, h = 0.f;
  int L = 0;
  if (active && !PACKED) {
    if (d.c0) c = d.c0[(long)b * n + j];
    if (d.h0) h = d.h0[(long)b * n + j];
    L = clamp_len(a.lens, b, T);
  }
  // The unit this thread publishes.  A unit is four consecutive units' h of one row (the tag is a bit of the fourth), and a
  // row's 32 units sit in 32 consecutive lanes, so the thread of every fourth unit takes its neighbours' values
  // through DPP shifts: no staging in shared memory, no second barrier.  m = which unit of the 16-unit tile (0..3).
  const int pp = u >> 4, m = (u & 15) >> 2;
  const int t16p = tile2 * 2 + pp;
  const int cch = t16p * 2 + (m >> 1);
  const long unit_index = (((long)rt * nkc + (cch >> 2)) * 64 + (cch & 3) * 16 + half * 8 + r8) * 2 + (m & 1);
  const bool publishes = (u & 3) == 0 && t16p < ntiles16;
  const bool local = group_is_xcd_local(a.xcc, wg.base, a.map.ntile, a.spin_limit);
  // Has this row had a frame yet?  Until then it publishes zeros, not the initial state it carries: that state's product
  // with W_h has been added to the pre-activations of the row's first frame by the host side, and what travels
  // through the ring must keep |h| <= 1 (the tag bit).
  bool started = false;

  // x W_x + b of a frame is read through a buffer descriptor that covers exactly that frame: a lane with nothing to
  // fetch (row past the batch, unit past n, frame past the row's length) has its offset parked outside and gets zeros
  // without touching memory, as does every lane once the frames are used up (zero-sized descriptor); of four units that end past
  // the frame the check drops those.  Nothing is predicated, so every step issues the same loads.
  // The outputs go the same way: one descriptor per array and frame (zero-sized if the array is absent), offsets
  // that never change, parked where a lane has nothing to store; and so does the ring store, whose descriptor ends
  // below the parking offset.  Frame sizes in bytes: gates [B,4n] float, y [B,ldy] bf16, cs [B,n] float, hprev [B,ldh] bf16.
  constexpr unsigned kParked = 0x7ff00000u;
  const unsigned g_bytes = (unsigned)B * 4u * n * 4u, y_bytes = (unsigned)B * d.ldy * 2u, s_bytes = (unsigned)B * n * 4u;
  const unsigned g_off = active ? ((unsigned)b * 4u * n + j) * 4u : kParked;
  const unsigned y_off = active ? ((unsigned)b * d.ldy + j) * 2u : kParked;
  const unsigned s_off = active ? ((unsigned)b * n + j) * 4u : kParked;
  const unsigned h_bytes = (unsigned)B * (unsigned)d.ldh * 2u, h_off = active ? ((unsigned)b * (unsigned)d.ldh + j) * 2u : kParked;
  const unsigned pub_off = publishes ? (unsigned)unit_index * 8u : kParked;
  // (rows one behind the other: one descriptor covers all frames - they end below the parking offset -, a lane's offset names its frame)
  auto frame_of = [&](const void* base, int t, unsigned bytes, bool present = true) {
    if constexpr (PACKED) return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, present && base != nullptr ? bytes * (unsigned)T : 0u, kBufFlags);
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (unsigned long long)(unsigned)t * bytes), 0, present && base != nullptr ? bytes : 0u, kBufFlags);
  };
  // The frames' values come from HBM, 450-530 ns away (1 us for the slowest of a group's 128 wavefronts), and a compute unit hands
  // loads back in the order of issue: ring loads asked for meanwhile wait for them.  With four loads a frame, one frame at a time,
  // that was a third of the step once the products took half their time (n = 1024, 32 rows, both directions: 2.18 us a step, 1.29
  // without the fetch, 1.34 with it from L2).  So a lane brings four units of one gate, a wavefront's two rows of a frame being ONE
  // load into LDS, and kAhead frames are fetched together: every other step pays, and hardly (2 frames: 1.40, 4: 1.51, 8: 1.45;
  // 256 units, 16 rows: 1.03, 1.16, 1.12).  With all of it the step went from 1.61 to 1.33 us (330 units, 21 rows: 1.24 to 0.96).
  const int zq = (lane >> 3) & 3, zu = tile2 * 32 + 4 * (lane & 7);
  const int L_row = b < B && zu < n ? clamp_len(a.lens, b, T) : 0;
  const unsigned zx_off = ((unsigned)b * 4u * n + (unsigned)zq * n + zu) * 4u;
  const unsigned zxs_wave = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&zxs[0][wave][0][0][0]);
  // (assembly: the compiler makes every later LDS read wait for all loads of this kind that it knows to be in flight)
  unsigned e_ahead[kAhead] = {};                           // table words of the frames that are fetched next
  auto look_ahead = [&](int tau0, int now) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < kAhead; ++f) e_ahead[f] = tab.at(tau0 + f, now);
  };
  auto fetch_zx = [&](int tau0) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < kAhead; ++f) {
      if constexpr (PACKED) {
        const unsigned e = e_ahead[f];
        const unsigned off = frame_off(e, 16u * n) + ((unsigned)zq * n + zu) * 4u;
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(zxs_wave + (unsigned)f * (unsigned)sizeof(zxs[0])), "v"((e & kRowValid) && zu < n ? off : kParked), "s"(frame_of(d.gates, 0, g_bytes)) : "memory");
        continue;
      }
      const bool ok = tau0 + f < T;
      const int t = d.rev ? T - 1 - tau0 - f : tau0 + f;
      const __amdgpu_buffer_rsrc_t rg =
          __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)d.gates + (unsigned long long)(unsigned)(ok ? t : 0) * g_bytes), 0, ok ? g_bytes : 0u, kBufFlags);
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(zxs_wave + (unsigned)f * (unsigned)sizeof(zxs[0])), "v"(t < L_row ? zx_off : kParked), "s"(rg) : "memory");
    }
  };
  unsigned h_prev_bits = pack_bf16x2(h, 0.f) & 0xffffu;     // what hprev receives: h before the step, as bf16
  tab.load(0);
  look_ahead(0, 0);
  fetch_zx(0);
  PROF_DECL
  auto step = [&](const int tau, auto parity) __attribute__((always_inline)) {
    float (&red_)[4][8][129] = red[decltype(parity)::value];
    const int t = d.rev ? T - 1 - tau : tau;
    const unsigned e = tab.at(tau, tau);
    const bool valid = active && (PACKED ? (e & kRowValid) != 0u : t < L);
    PROF_MARK(4)
    const uint4* rin = ((tau & 1) ? d.ring1 : d.ring0) + (long)rt * nkc * 64;
    uint4* rout = (tau & 1) ? d.ring0 : d.ring1;
    const auto rd = [&]() __attribute__((always_inline)) {
      const unsigned tag = ll_fwd_tag((unsigned)tau) << 14;
      if constexpr (PACKED) return make_reader_pairs<NL>(rin, nkc, ntiles16 * 2, wave, lane, half, tag, err, a.spin_limit, rot);
      else return make_reader_half(rin, nkc, ntiles16 * 2, wave, lane, half, tag, err, a.spin_limit, rot);
    }();
    constexpr int zslot = decltype(parity)::value;
    constexpr bool fetches = zslot == kAhead - 1;
    float zx[4];
    auto fetch_next = [&]() __attribute__((always_inline)) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // the last of the frames has been read
      fetch_zx(tau + 1);
    };
    f32x4 acc[4];
    {
      auto use_single = [&](int p, const u32x4& raw) {     // a load fetched again after the stream, tags still in it
        u32x4 av[2];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const unsigned v = raw[c] & ((c & 1) ? ~kLLFwdTagBit : ~0u);
          av[0][c] = rows_from_low(v);
          av[1][c] = rows_from_high(v);
        }
        operands_settle(av[0], av[1]);
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
          for (int q = 0; q < 4; ++q) smfmac_b_agpr(acc[q], av[o], w[2 * p + o][q], sparse);
      };
      // The stream.  The loads are consumed in pairs (the last one alone where NL is odd): a pair is four chunks, and every accumulator takes its four products in that
      // order.  A product of this shape issues every 16 cycles (7.05 ns measured, in any order of the
      // accumulators) and occupies the issue slot of the wavefront for 4 of them: independent instructions behind
      // it are free, dependent ones are not (three: 12.4 ns).  What turns the loads
      // into operands (tag test, masking the tags off, chunks into all rows) is cut into single instructions that follow the
      // products of the chunk before.  A pair with a stale tag in any lane is skipped (wave-uniform branch)
      // and both its loads are fetched again by fix_up.
      constexpr int NP = (NL + 1) / 2;
      u32x4 x[NL];
      const unsigned tagw = rd.tag << 16;
      // The poll IS the first pair of loads: they are repeated (bounded) until all their tags have turned, and what
      // the last round fetched is kept.  Only then are the other loads issued; their round trip passes behind the
      // first pair's MFMAs instead of in front of the whole stream (a poll of its own followed by all loads cost one
      // round trip more per step, a tenth of it).  (Nine times out of ten the first round succeeds; yet issuing
      // everything at once without looking was measured slower: the values arrive while the poll is in flight.)
      auto poll_loads = [&]() __attribute__((always_inline)) {
        x[0] = rd.load_it(rd.it_of(0));
        if constexpr (NL > 1) x[1] = rd.load_it(rd.it_of(1));
      };
      auto polled_stale = [&]() __attribute__((always_inline)) {
        unsigned stale = rd.tag_diff(x[0], rd.it_of(0), tagw);
        if constexpr (NL > 1) stale |= rd.tag_diff(x[1], rd.it_of(1), tagw);
        return __builtin_amdgcn_ballot_w64(stale > 0xffffu) != 0ull;
      };
      poll_loads();
      // The accumulators are cleared while the poll is in flight.  (By moves: starting each chain with an MFMA that
      // adds to the constant 0, as the 16-row backward kernel does, was measured 10 % slower per step here.)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
      operands_settle(acc[0], acc[1], acc[2], acc[3]);
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(polled_stale() && !dead, 0)) rd.poll_again(dead, poll_loads, polled_stale);
      PROF_MARK(5)
      __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0): nothing is in flight behind the poll, frames included
#pragma unroll
      for (int i = 2; i < NL; ++i) x[i] = rd.load_it(rd.it_of(i));
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int q = 0; q < 4; ++q) zx[q] = zxs[zslot][wave][lane >> 5][q][u];
      if (PACKED && fetches) look_ahead(tau + 1, tau);
      __builtin_amdgcn_sched_barrier(0);
      u32x4 ops[NL][2];
      unsigned bad[NP];                                    // tag mismatches of the pair, per lane, in the upper 16 bits
      // step 0: tag test; 1, 2: tags off; 3 .. 6: first chunk into all rows; 7 .. 10: second chunk
      auto prep = [&](int i, int kk) __attribute__((always_inline)) {
        if (kk == 0) {
          const unsigned m = rd.tag_diff(x[i], rd.it_of(i), tagw);
          bad[i >> 1] = (i & 1) ? (bad[i >> 1] | m) : m;
        } else if (kk < 3) {
          x[i][2 * kk - 1] &= ~kLLFwdTagBit;
        } else if (kk < 7) {
          ops[i][0][kk - 3] = rows_from_low(x[i][kk - 3]);
        } else {
          ops[i][1][kk - 7] = rows_from_high(x[i][kk - 7]);
        }
      };
      unsigned long long redo = 0ull;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        __builtin_amdgcn_sched_barrier(0);
        const bool two = 2 * p + 1 < NL;
        if (p > 0) { prep(2 * p, 0); if (two) prep(2 * p + 1, 0); }      // (the poll has looked at the first pair)
        if (p == 0 || __builtin_expect(__builtin_amdgcn_ballot_w64(bad[p] > 0xffffu) == 0ull, 1)) {
#pragma unroll
          for (int kk = 1; kk < 7; ++kk) prep(2 * p, kk);
          operands_settle(ops[2 * p][0]);
          // The next frames go out where this wavefront's last ring load has arrived: the compute unit hands loads back in the
          // order of issue, other wavefronts' included, so earlier they hold up ring loads still in flight, and later they are in the
          // next step's poll's way.
          if (fetches && p == NP - 1 && redo == 0ull) fetch_next();
#pragma unroll
          for (int o = 0; o < (two ? 4 : 2); ++o)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              smfmac_b_agpr(acc[q], ops[2 * p + (o >> 1)][o & 1], w[4 * p + o][q], sparse);
              __builtin_amdgcn_sched_barrier(0);
              // the pair's other operands, two products ahead of theirs (the wait states between the two)
              const int i = 2 * p + (o > 0), kk = o == 1 ? 3 : 7;
              if (o < (two ? 3 : 1) && q < 2) { prep(i, kk + 2 * q); prep(i, kk + 2 * q + 1); }
              if (two && o == 0 && q == 2) { prep(i + 1, 1); prep(i + 1, 2); }
              __builtin_amdgcn_sched_barrier(0);
            }
        } else {                                           // rare once the sample has turned
          redo |= (two ? 3ull : 1ull) << (2 * p);
        }
      }
      PROF_REDO(__popcll(redo))
      const bool asked_again = redo != 0ull;
      if (redo) {
        rd.template fix_up_batch<NL>(redo, dead, use_single);
        // (nothing of that is outstanding any more - said with an instruction the compiler takes note of: it cannot tell
        // from the loop's exits, and would make whatever reuses those registers below wait for every load in flight)
        __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0)
      }
      mfma_settle(acc[0], acc[1], acc[2], acc[3]);
      if (fetches && asked_again) fetch_next();
    }
    PROF_MARK(0)
    // fragment rows 4*(lane/16) + v: rows 0-7 of the unit tile's first 16 columns, then of the others
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) red_[wave][4 * ((lane >> 4) & 1) + v][q * 32 + (lane >> 5) * 16 + (lane & 15)] = acc[q][v];
    PROF_MARK(1)
    __syncthreads();

    if constexpr (PACKED) {
      if ((e & kRowFirst) && active) {
        c = 0.f; h = 0.f;
        if (d.c0 || d.h0) {
          const long s0 = (long)((e & kRowFrame) % (unsigned)B) * n + j;
          if (d.c0) c = rare_load(&d.c0[s0]);
          if (d.h0) h = rare_load(&d.h0[s0]);
        }
        h_prev_bits = pack_bf16x2(h, 0.f) & 0xffffu;
      }
    }
    CellOut o = {};
    if (valid) {
      float zh[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) zh[q] = red_[0][r8][q * 32 + u] + red_[1][r8][q * 32 + u] + red_[2][r8][q * 32 + u] + red_[3][r8][q * 32 + u];
      o = lstm_cell(zh, zx, c);
      c = o.c; h = o.h;
    }
    const unsigned h_bits = pack_bf16x2(h, 0.f) & 0xffffu; // inactive threads hold h = 0: padding rows / units publish zeros
    started = PACKED ? valid && !(e & kRowLast) : started || valid;
    PROF_MARK(2)
    {                                 // the recurrence's critical store goes out first
      // h of the next three units of the tile (DPP row_shl:1, :2, :3; past the row of 16 lanes: zero)
      const unsigned x0 = started ? h_bits : 0u;
      const unsigned x1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x101, 0xf, 0xf, true);
      const unsigned x2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x102, 0xf, 0xf, true);
      const unsigned x3 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x103, 0xf, 0xf, true);
      const u32x2 unit = {x0 | (x1 << 16), x2 | (x3 << 16) | (ll_fwd_tag((unsigned)tau + 1u) << 30)};
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)((tau & 1) ? d.ring0 : d.ring1), 0, kParked, kBufFlags);
      // 1: workgroup scope, stays in this XCD's L2;  16: agent scope, written through
      if (local) __builtin_amdgcn_raw_buffer_store_b64(unit, ro, pub_off, 0, 1);
      else __builtin_amdgcn_raw_buffer_store_b64(unit, ro, pub_off, 0, 16);
    }
    {                                 // layer outputs and what the backward pass needs (2: non-temporal)
      // (padded frames are filled by a launch of its own where rows run one behind the other)
      const unsigned yo = PACKED ? (valid ? frame_off(e, 2u * (unsigned)d.ldy) + 2u * j : kParked) : y_off, so = PACKED ? (valid ? frame_off(e, 4u * n) + 4u * j : kParked) : s_off;
      const unsigned ho = PACKED ? (valid ? frame_off(e, 2u * (unsigned)d.ldh) + 2u * j : kParked) : h_off;
      __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(valid ? h_bits : 0u), frame_of(d.y, t, y_bytes), yo, 0, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c), frame_of(d.cs, t, s_bytes), so, 0, 2);
      __builtin_amdgcn_raw_buffer_store_b16((unsigned short)h_prev_bits, frame_of(d.hprev, t, h_bytes), ho, 0, 2);
      const __amdgpu_buffer_rsrc_t rw = frame_of(d.gates, t, g_bytes, a.write_gates != 0);
      const unsigned gw = valid ? (PACKED ? frame_off(e, 16u * n) + 4u * j : g_off) : kParked;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o.gi), rw, gw, 0u, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o.gf), rw, gw, 4u * n, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o.gg), rw, gw, 8u * n, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o.go), rw, gw, 12u * n, 2);
    }
    if constexpr (PACKED) {
      if ((e & kRowLast) && active && (d.cT || d.hT)) {
        const long s0 = (long)((e & kRowFrame) % (unsigned)B) * n + j;
        if (d.cT) d.cT[s0] = c;
        if (d.hT) d.hT[s0] = h;
      }
    }
    h_prev_bits = h_bits;
    PROF_MARK(3)
  };
  for (int tau = 0; tau < tab.steps; tau += 2) {
    if (PACKED && tau > 0 && (tau & (kTabSteps - 1)) == 0) tab.load(tau);
    step(tau, std::integral_constant<int, 0>{});
    if (tau + 1 < tab.steps) step(tau + 1, std::integral_constant<int, 1>{});
  }
  PROF_DUMP("fwd8", T)
  if constexpr (PACKED) {
    if (wg.rt == 0 && active && (d.cT || d.hT))            // rows without frames keep their state
      for (int bb = r8; bb < B; bb += 8)
        if (clamp_len(a.lens, bb, T) == 0) {
          const long s0 = (long)bb * n + j;
          if (d.cT) d.cT[s0] = d.c0 ? d.c0[s0] : 0.f;
          if (d.hT) d.hT[s0] = d.h0 ? d.h0[s0] : 0.f;
        }
  } else if (active) {
    if (d.cT) d.cT[(long)b * n + j] = c;
    if (d.hT) d.hT[(long)b * n + j] = h;
  }
}

// ------------------------------------------------------------------------------------------------
// forward, third decomposition: a work-group owns 32 units for all 16 rows of a row tile.  For batches of more than
// 32 rows: 64 rows x 2 directions are then 256 work-groups, one launch, where the 32 x 8 form needs two launches
// that each walk all T steps.  Every MFMA row is a real row (96 MFMAs per wavefront and step, as in the 32 x 8 form,
// for twice the rows), a load is one whole chunk (12 loads per wavefront and step instead of 6), and a thread
// updates two cells (rows r8 and r8 + 8).  Ring layout, tags and publishing are those of the 32 x 8 form.
template <int NIT> struct Fwd16Lds {
  alignas(16) float red[2][4][16][129];                  // two copies, used by even and odd steps: one barrier per step
  // x W_x + b of the next frames, fetched two together (see the 32 x 8 kernel): [frame][row half][wavefront][row][gate][unit], a
  // wavefront reading back what it asked for, so no barrier is involved - only the loads' completion.
  alignas(16) float zxs[2][2][4][2][4][32];
  u32x4 rbuf[4][NIT][64];                                // the ring loads of a step: [wavefront][load][lane], written by the memory unit
};
template <int NIT>
__device__ __forceinline__ void fwd16_body(const PFwdArgs& a, const GridMap& map, Fwd16Lds<NIT>& lds) {
  auto& red = lds.red;
  auto& zxs = lds.zxs;
  auto& rbuf = lds.rbuf;
  const WgCoord wg = wg_coord(map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const PFwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int tile2 = wg.tile, rt = a.rt0 + wg.rt;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // (told to be wave-uniform: it forms scalar LDS addresses below)
  const int nkc = a.nkc, n = a.n, B = a.B, T = a.T;
  const int ntiles16 = (n + 15) / 16;
  unsigned* err = a.sync;
  bool dead = false;

  const int nitv = (nkc + 3) / 4, rot = tile2 % nitv;
  // Register set `it` holds the chunk that load `it` of the stream fetches; the first kAccIts sets fill the 256
  // accumulation registers, the rest sit in vector registers (as in the 32 x 8 form).
  constexpr int kAccIts = NIT < 8 ? NIT : 8;
  u32x4 wa[kAccIts][2][4];
  u32x4 wv[NIT - kAccIts > 0 ? NIT - kAccIts : 1][2][4];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int kc = wave + 4 * rot_index(it, rot, nitv);
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int t16 = tile2 * 2 + ct;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4* src = (kc < nkc && t16 < ntiles16) ? &d.Wf[((long)(t16 * 4 + q) * nkc + kc) * 64 + lane] : &d.Wzero[lane];
        if (it < kAccIts) wa[it][ct][q] = load_to_agpr(src);
        else wv[it - kAccIts][ct][q] = *(const u32x4*)src;
      }
    }
  }
  agpr_loads_done();

  const int r8 = tid >> 5, u = tid & 31;                 // pointwise pairs of this thread: rows r8 and r8 + 8, unit u of 32
  const int j = tile2 * 32 + u;
  float c[2] = {0.f, 0.f}, h[2] = {0.f, 0.f};
  int L[2] = {0, 0};
  bool active[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = rt * 16 + r8 + 8 * k;
    active[k] = b < B && j < n;
    if (active[k]) {
      if (d.c0) c[k] = d.c0[(long)b * n + j];
      if (d.h0) h[k] = d.h0[(long)b * n + j];
      L[k] = clamp_len(a.lens, b, T);
    }
  }
  const int pp = u >> 4, m = (u & 15) >> 2;                // the unit (four units' h, see the 32 x 8 kernel) this thread publishes
  const int t16p = tile2 * 2 + pp;
  const int cch = t16p * 2 + (m >> 1);
  const bool publishes = (u & 3) == 0 && t16p < ntiles16;
  bool started[2] = {false, false};                      // (see the 32 x 8 kernel)
  const bool local = group_is_xcd_local(a.xcc, wg.base, a.map.ntile, a.spin_limit);

  constexpr unsigned kParked = 0x7ff00000u;
  const unsigned g_bytes = in_sgpr((unsigned)B * 4u * n * 4u), y_bytes = in_sgpr((unsigned)B * d.ldy * 2u), s_bytes = in_sgpr((unsigned)B * n * 4u);
  // offsets of row r8 inside a frame; row r8 + 8 lies a wave-uniform distance behind it (a row of the second half
  // that exists implies its partner in the first half does), which keeps four registers free
  const unsigned b0 = (unsigned)(rt * 16 + r8);
  const unsigned g_off0 = active[0] ? (b0 * 4u * n + j) * 4u : kParked;
  const unsigned y_off0 = active[0] ? (b0 * d.ldy + j) * 2u : kParked;
  const unsigned s_off0 = active[0] ? (b0 * n + j) * 4u : kParked;
  const unsigned h_bytes = (unsigned)B * (unsigned)d.ldh * 2u, h_off0 = active[0] ? (b0 * (unsigned)d.ldh + j) * 2u : kParked;
  const unsigned pub_off0 = publishes ? (unsigned)((((long)rt * nkc + (cch >> 2)) * 64 + (cch & 3) * 16 + r8) * 2 + (m & 1)) * 8u : kParked;
  auto g_off = [&](int k) { return k == 0 ? g_off0 : (active[1] ? g_off0 + 8u * 4u * n * 4u : kParked); };
  auto y_off = [&](int k) { return k == 0 ? y_off0 : (active[1] ? y_off0 + 8u * (unsigned)d.ldy * 2u : kParked); };
  auto s_off = [&](int k) { return k == 0 ? s_off0 : (active[1] ? s_off0 + 8u * n * 4u : kParked); };
  auto h_off = [&](int k) { return k == 0 ? h_off0 : (active[1] ? h_off0 + 8u * (unsigned)d.ldh * 2u : kParked); };
  auto pub_off = [&](int k) { return k == 0 ? pub_off0 : (publishes ? pub_off0 + 8u * 16u : kParked); };
  auto frame_of = [&](const void* base, int t, unsigned bytes, bool present = true) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (unsigned long long)(unsigned)t * bytes), 0, present && base != nullptr ? bytes : 0u, kBufFlags);
  };
  const unsigned zxs_wave = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&zxs[0][0][wave][0][0][0]);
  const unsigned rbuf_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&rbuf[0][0][0];
  const int zu = tile2 * 32 + 4 * (lane & 7);
  int L_row[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) L_row[k] = (int)b0 + 8 * k < B && zu < n ? clamp_len(a.lens, b0 + 8 * k, T) : 0;
  const unsigned zx_off = (b0 * 4u * n + ((unsigned)lane >> 3 & 3u) * n + zu) * 4u;
  // (assembly: the compiler makes every later LDS read wait for all loads of this kind that it knows to be in flight)
  auto fetch_zx = [&](int tau0) __attribute__((always_inline)) {      // frames of steps tau0 and tau0 + 1
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const bool ok = tau0 + f < T;
      const int t = d.rev ? T - 1 - tau0 - f : tau0 + f;
      const __amdgpu_buffer_rsrc_t rg =
          __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)d.gates + (unsigned long long)(unsigned)(ok ? t : 0) * g_bytes), 0, ok ? g_bytes : 0u, kBufFlags);
#pragma unroll
      for (int k = 0; k < 2; ++k)
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(zxs_wave + (unsigned)(f * sizeof(zxs[0]) + k * sizeof(zxs[0][0]))),
                     "v"(t < L_row[k] ? zx_off : kParked), "s"(rg), "s"((unsigned)k * 8u * 4u * n * 4u) : "memory");
    }
  };
  unsigned h_prev_bits[2] = {pack_bf16x2(h[0], 0.f) & 0xffffu, pack_bf16x2(h[1], 0.f) & 0xffffu};
  fetch_zx(0);
  PROF_DECL
  auto step = [&](const int tau, auto parity) __attribute__((always_inline)) {
    constexpr int kSet = decltype(parity)::value;
    float (&red_)[4][16][129] = red[decltype(parity)::value];
    const int t = d.rev ? T - 1 - tau : tau;
    PROF_MARK(4)
    const uint4* rin = ((tau & 1) ? d.ring1 : d.ring0) + (long)rt * nkc * 64;
    RingReader rd = make_reader(rin, nkc, ntiles16 * 2, wave, lane, ll_fwd_tag((unsigned)tau) << 14, err, a.spin_limit, rot);
    f32x4 acc[2][4];
    float zx_[2][4];
    {
      auto mma_one = [&](int it, int ct, int q, const u32x4& a_op) __attribute__((always_inline)) {
        if (it < kAccIts) mfma_b_agpr(acc[ct][q], a_op, wa[it < kAccIts ? it : 0][ct][q]);
        else mfma_b_vgpr(acc[ct][q], a_op, wv[it >= kAccIts ? it - kAccIts : 0][ct][q]);
      };
      auto use_single = [&](int i, const u32x4& raw) {     // a load fetched again after the stream, tags still in it
        u32x4 av = {raw[0], raw[1] & ~kLLFwdTagBit, raw[2], raw[3] & ~kLLFwdTagBit}, dummy = av;
        operands_settle(av, dummy);
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int q = 0; q < 4; ++q) mma_one(i, ct, q, av);
      };
      // The loads are consumed in pairs (two chunks, 16 MFMAs); what turns the next pair's loads into operands (tag
      // test, masking the tags off) is cut into single instructions that follow the first MFMAs of the pair before.
      static_assert(NIT % 2 == 0, "loads are consumed in pairs");
      constexpr int NP = NIT / 2, kPrepSteps = 6;
      // The first pair of loads is the poll and lands in registers.  The others are written to LDS by the memory
      // unit (rbuf: no registers are held while they are in flight, so all of them fly at once) and are read back
      // a pair ahead of their MFMAs; loads complete in the order of issue, which is what the counted waits rely on.
      u32x4 x[2][2];
      const unsigned tagw = rd.tag << 16;
      auto issue_dma = [&](int i) __attribute__((always_inline)) {
        const unsigned dst = rbuf_base + (unsigned)(wave * NIT + i) * 1024u, soff = (unsigned)rd.it_of(i) * rd.it_bytes;
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen sc1 lds" ::"s"(dst), "v"(rd.voff), "s"(rd.rs), "s"(soff) : "memory");
      };
      // (Fetching everything along with the first poll - stale loads now being cheap to repeat - was measured 15 % slower
      // per step: the polled pair then returns behind 10 KiB of other loads, most of which are repeated anyway.)
      auto poll_loads = [&]() __attribute__((always_inline)) {
        x[0][0] = rd.load_it(rd.it_of(0));
        x[0][1] = rd.load_it(rd.it_of(1));
      };
      auto polled_stale = [&]() __attribute__((always_inline)) {
        const unsigned stale = rd.tag_diff(x[0][0], rd.it_of(0), tagw) | rd.tag_diff(x[0][1], rd.it_of(1), tagw);
        return __builtin_amdgcn_ballot_w64(stale > 0xffffu) != 0ull;
      };
      poll_loads();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[ct][q] = (f32x4){0.f, 0.f, 0.f, 0.f};
      operands_settle(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
      operands_settle(acc[1][0], acc[1][1], acc[1][2], acc[1][3]);
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(polled_stale() && !dead, 0)) rd.poll_again(dead, poll_loads, polled_stale);
      PROF_MARK(5)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing is in flight behind the poll, frames included
#pragma unroll
      for (int i = 2; i < NIT; ++i) issue_dma(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) zx_[k][q] = zxs[kSet][k][wave][lane >> 5][q][u];
      __builtin_amdgcn_sched_barrier(0);
      unsigned bad[NP];
      // pair p + 1 becomes operands behind MFMA `at` of pair p: wait for its loads, read them from LDS (step -1);
      // tag test and masking (steps 0 .. kPrepSteps - 1) follow a few MFMAs later, when the LDS reads have returned
      auto prep = [&](auto P, int k) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value;
        u32x4 (&xp)[2] = x[p & 1];
        if (k < 0) {
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NIT - 2 - 2 * p) : "memory");     // all but the loads behind this pair have landed
          xp[0] = rbuf[wave][2 * p][lane];
          xp[1] = rbuf[wave][2 * p + 1][lane];
          return;
        }
        const int second = k >= kPrepSteps / 2, i = 2 * p + second, kk = second ? k - kPrepSteps / 2 : k;
        u32x4& xi = xp[second];
        if (kk == 0) {
          const unsigned mm = rd.tag_diff(xi, rd.it_of(i), tagw);
          bad[p] = second ? (bad[p] | mm) : mm;
        } else if (kk == 1) {
          xi[1] &= ~kLLFwdTagBit;
        } else {
          xi[3] &= ~kLLFwdTagBit;
        }
      };
      unsigned long long redo = 0ull;
      bool zx_asked = false;
#pragma unroll
      for (int k = 0; k < kPrepSteps; ++k) prep(std::integral_constant<int, 0>{}, k);
      static_for<NP>([&](auto P) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value;
        constexpr std::integral_constant<int, (p + 1 < NP ? p + 1 : p)> P1{};
        // the second pair's loads have just been issued: reading them early would only stall this pair's MFMAs
        constexpr int read_at = p == 0 ? 15 : 2, prep_at = p == 0 ? 16 : 9;
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad[p] > 0xffffu) == 0ull, 1)) {
          operands_settle(x[p & 1][0], x[p & 1][1]);
          // The next frame's x W_x + b goes out where this wavefront's last ring load has arrived (see the 32 x 8 kernel) -
          // unless a pair is being fetched again: the second look below waits for everything in flight, and these come from HBM.
          if (kSet == 1 && p == NP - 1 && redo == 0ull) {
            fetch_zx(tau + 1);
            zx_asked = true;
          }
#pragma unroll
          for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                mma_one(2 * p + o, ct, q, x[p & 1][o]);
                const int mm = (o * 2 + ct) * 4 + q;
                if (p + 1 < NP && (mm == read_at || (mm >= prep_at && mm < prep_at + kPrepSteps))) {
                  __builtin_amdgcn_sched_barrier(0);
                  prep(P1, mm == read_at ? -1 : mm - prep_at);
                  __builtin_amdgcn_sched_barrier(0);
                }
              }
          if (p + 1 < NP) {
#pragma unroll
            for (int k = 0; k < kPrepSteps; ++k)
              if (prep_at + k >= 16) prep(P1, k);            // what did not fit behind this pair's MFMAs
          }
        } else {
          // Stale: the pair's loads are issued again at once, behind the others, and looked at after the last pair, so
          // their round trip passes behind the MFMAs still to come.  (The counted waits of later pairs then wait for
          // up to that many loads more than they need: loads complete in order, so they wait for no less.)
          redo |= 3ull << (2 * p);
          if (p > 0) {
            issue_dma(2 * p);
            issue_dma(2 * p + 1);
          }
          if (p + 1 < NP) {
#pragma unroll
            for (int k = -1; k < kPrepSteps; ++k) prep(P1, k);
          }
        }
      });
      if (redo >> 2) {                                     // the second look at what was fetched again
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        static_for<NP - 1>([&](auto P) __attribute__((always_inline)) {
          constexpr int p = decltype(P)::value + 1;
          if ((redo >> (2 * p)) & 1ull) {
            const u32x4 y0 = rbuf[wave][2 * p][lane], y1 = rbuf[wave][2 * p + 1][lane];
            if (__builtin_amdgcn_ballot_w64((rd.stale_bits(y0, rd.it_of(2 * p)) | rd.stale_bits(y1, rd.it_of(2 * p + 1))) != 0u) == 0ull) {
              use_single(2 * p, y0);
              use_single(2 * p + 1, y1);
              redo &= ~(3ull << (2 * p));
            }
          }
        });
      }
      PROF_REDO(__popcll(redo))
      if (redo) {                                          // (a quarter of the loads at a time: registers)
        rd.template fix_up_batch<NIT / 4, 0>(redo, dead, use_single);
        rd.template fix_up_batch<NIT / 4, NIT / 4>(redo, dead, use_single);
        rd.template fix_up_batch<NIT / 4, NIT / 2>(redo, dead, use_single);
        rd.template fix_up_batch<NIT / 4, 3 * (NIT / 4)>(redo, dead, use_single);
      }
      mfma_settle(acc[0][0], acc[0][1], acc[0][2], acc[0][3], acc[1][0], acc[1][1], acc[1][2], acc[1][3]);
      if (kSet == 1 && !zx_asked) fetch_zx(tau + 1);
    }
    PROF_MARK(0)
    // (LDS addresses are formed anew in every step: hoisted out of the loop they stay in registers the loop does not have)
    int lane_ = lane, u_ = u, r8_ = r8;
    asm volatile("" : "+v"(lane_), "+v"(u_), "+v"(r8_));
    // accumulator rows 4*(lane/16) + v: every row is one of this work-group's
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) red_[wave][4 * (lane_ >> 4) + v][q * 32 + ct * 16 + (lane_ & 15)] = acc[ct][q][v];
    PROF_MARK(1)
    __syncthreads();
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)((tau & 1) ? d.ring0 : d.ring1), 0, kParked, kBufFlags);
    const __amdgpu_buffer_rsrc_t ry = frame_of(d.y, t, y_bytes), rc = frame_of(d.cs, t, s_bytes), rh = frame_of(d.hprev, t, h_bytes);
    const __amdgpu_buffer_rsrc_t rw = frame_of(d.gates, t, g_bytes, a.write_gates != 0);
    // both cells first, then both ring stores (the recurrence's critical stores, close together so that the two halves
    // of a row tile turn their tags at about the same time), then the outputs
    CellOut o[2] = {};
    bool valid[2];
    unsigned h_bits[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int rr = r8_ + 8 * k;
      valid[k] = active[k] && t < L[k];
      if (valid[k]) {
        float zh[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) zh[q] = red_[0][rr][q * 32 + u_] + red_[1][rr][q * 32 + u_] + red_[2][rr][q * 32 + u_] + red_[3][rr][q * 32 + u_];
        float zx[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) zx[q] = zx_[k][q];
        o[k] = lstm_cell(zh, zx, c[k]);
        c[k] = o[k].c; h[k] = o[k].h;
      }
      h_bits[k] = pack_bf16x2(h[k], 0.f) & 0xffffu;         // inactive threads hold h = 0: padding rows / units publish zeros
      started[k] = started[k] || valid[k];
    }
    PROF_MARK(2)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const unsigned x0 = started[k] ? h_bits[k] : 0u;
      const unsigned x1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x101, 0xf, 0xf, true);
      const unsigned x2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x102, 0xf, 0xf, true);
      const unsigned x3 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x0, 0x103, 0xf, 0xf, true);
      const u32x2 unit = {x0 | (x1 << 16), x2 | (x3 << 16) | (ll_fwd_tag((unsigned)tau + 1u) << 30)};
      if (local) __builtin_amdgcn_raw_buffer_store_b64(unit, ro, pub_off(k), 0, 1);
      else __builtin_amdgcn_raw_buffer_store_b64(unit, ro, pub_off(k), 0, 16);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {          // layer outputs and what the backward pass needs (2: non-temporal)
      __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(valid[k] ? h_bits[k] : 0u), ry, y_off(k), 0, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c[k]), rc, s_off(k), 0, 2);
      __builtin_amdgcn_raw_buffer_store_b16((unsigned short)h_prev_bits[k], rh, h_off(k), 0, 2);
      const unsigned gw = valid[k] ? g_off(k) : kParked;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[k].gi), rw, gw, 0u, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[k].gf), rw, gw, 4u * n, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[k].gg), rw, gw, 8u * n, 2);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[k].go), rw, gw, 12u * n, 2);
      h_prev_bits[k] = h_bits[k];
    }
    PROF_MARK(3)
  };
  for (int tau = 0; tau < T; tau += 2) {
    step(tau, std::integral_constant<int, 0>{});
    if (tau + 1 < T) step(tau + 1, std::integral_constant<int, 1>{});
  }
  PROF_DUMP("fwd16r", T)
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = rt * 16 + r8 + 8 * k;
    if (active[k]) {
      if (d.cT) d.cT[(long)b * n + j] = c[k];
      if (d.hT) d.hT[(long)b * n + j] = h[k];
    }
  }
}

// ------------------------------------------------------------------------------------------------
// backward, third decomposition ("partial sums"): no dz crosses work-groups.  A work-group still owns 32 units for
// 8 rows, but it multiplies ITS dz (8 rows x 128 gate columns) by the matching 128 rows of W_h^T for ALL n outputs
// and publishes, per destination tile of 32 units, a partial sum of Dh (bf16).  A consumer adds the partial sums
// of its tile from all producers: 1 KiB per producer, 32 KiB per step at n = 1024, where reading dz itself takes
// 88 KiB.  The ring read is what bounds the backward step, so this is the fastest of the three forms.  Dh is
// therefore a sum of bf16-rounded partial sums (accumulated in float), not a float product of bf16-rounded dz.
//
// With one wavefront per SIMD every instruction's latency is exposed (about 2 ns each), so the formats are chosen
// to keep instruction counts low: an 8-byte unit holds values of ONE output for four ROWS, which
// is how an MFMA accumulator lane holds them, so a producer stores straight from its accumulators - no staging,
// no cross-lane moves.  (n = 1024, 32 rows, both directions: 1.75 us a step with dense products that compute every row twice and
// inputs fetched a frame at a time, 1.33 now; 330 units, 21 rows 1.41, 1.03.)  Ring layout per direction and slot:
//   [row group][destination tile][producer tile][32 outputs][2 row halves] x 8 bytes (rows 4g .. 4g+3 as bf16).
// The tag is ONE BIT, bit 14 of the fourth value (see the forward ring): the partial sums travel scaled by 2^-32 - the
// packed W_h carries the factor, so the MFMAs deliver them scaled, and the consumer multiplies its sum by 2^32 - which
// leaves that bit 0 for every partial sum below 2^33 in magnitude and changes no other bit of any value above 2^-94
// (a power of two commutes with every rounding on the way).  A partial sum of 2^33 or more cannot be exchanged: its
// unit looks stale or fresh at random; gradients of that size are past use, and the case mostly ends in an expired wait.
// Half the bytes and half the ring loads of the format this replaces (3 values + a 16-bit tag per unit, 16 bytes per lane).
// W_h slice in registers: w[kc][c] = B fragment of gate kc (K = this tile's 32 units) for column tile
// wave*16 + c of the n outputs.
constexpr int kPartBytes = 512;                           // one (producer, destination tile)
constexpr float kPartScale = 1.f / 4294967296.f;          // 2^-32
// tag bit of the partial sums that backward step sigma (= T-1-tau) consumes: written by step sigma - 1 into slot
// (sigma - 1) & 1; alternates between consecutive uses of a slot and is 1 at the first, so zero-filled slots look unwritten
__device__ __forceinline__ unsigned part_tag(int sigma) { return ((((unsigned)sigma - 1u) >> 1) & 1u) ^ 1u; }

template <int NCT, bool PACKED> struct Bwd8Lds {
  static constexpr int kAhead = NCT == 16 ? 2 : 4;       // frames whose inputs are fetched together (fetch_in below)
  static_assert(kAhead >= 2, "a step reads its inputs before its poll: they have to be there from the step before");
  alignas(16) float red[8][8][33];                       // [wavefront, producer of the pair][row][output]
  alignas(16) unsigned short zb[8][136];
  // inputs of the next frames, [frame][wavefront][...][lane or row, unit]: a wavefront reads back what it asked for
  alignas(16) float in_g[2 * kAhead][4][2][4][32];
  alignas(16) float in_c[2 * kAhead][4][64];
  alignas(16) unsigned in_y[2 * kAhead][4][64];
  alignas(16) float in_n[PACKED ? 2 * kAhead : 1][4][64];
  alignas(16) unsigned tab[RowTable<PACKED>::kSteps][8];
  float dbred[8][129];
};
template <int NPW, int NCT, bool PACKED>                  // n <= 128 * NPW (producers per wavefront) and n <= 64 * NCT (its output column tiles)
__device__ __forceinline__ void bwd8_body(const PBwdArgs& a, Bwd8Lds<NCT, PACKED>& lds) {
  constexpr int kAhead = Bwd8Lds<NCT, PACKED>::kAhead;
  auto& red = lds.red;
  auto& zb = lds.zb;
  auto& in_g = lds.in_g;
  auto& in_c = lds.in_c;
  auto& in_y = lds.in_y;
  auto& in_n = lds.in_n;
  auto& tab_lds = lds.tab;
  const WgCoord wg = wg_coord(a.map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const PBwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int J = wg.tile, R = 2 * a.rt0 + wg.rt, ntile2 = a.map.ntile;     // R: row group of 8 rows, counted over the whole batch
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int n = a.n, B = a.B, T = a.T;
  unsigned* err = a.sync;
  bool dead = false;

  u32x4 w4[4][NCT / 2][2];                               // all 256 accumulation registers at NCT = 16
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
#pragma unroll
    for (int P = 0; P < NCT / 2; ++P)
#pragma unroll
      for (int set = 0; set < 2; ++set) w4[kc][P][set] = load_to_agpr(&d.Wb[((((long)J * 4 + wave) * 4 + kc) * NCT + 2 * P + set) * 64 + lane]);
  agpr_loads_done();
  u32x8 w[4][NCT / 2];                                   // gate kc, destination tile P of this wavefront (two column tiles)
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
#pragma unroll
    for (int P = 0; P < NCT / 2; ++P) w[kc][P] = agpr_join(w4[kc][P][0], w4[kc][P][1]);
  const int sparse = (lane & 8) ? kSparseHigh : kSparseLow;

  const int r8 = tid >> 5, u = tid & 31;                 // pointwise pair of this thread
  const int b = PACKED ? 0 : R * 8 + r8, j = J * 32 + u;
  const bool active = b < B && j < n;
  const RowTable<PACKED> tab = {tab_lds, PACKED ? d.tab + (long)wg.rt * a.tab_steps * 8 : nullptr, PACKED ? __builtin_amdgcn_readfirstlane(a.steps[wg.rt]) : T, r8};
  const int Tn = tab.steps;                                // backward steps
  unsigned e_prev = 0u;                                    // (rows one behind the other) the step before
  float Dh = 0.f, Dc = 0.f;
  float dbsum[4] = {0.f, 0.f, 0.f, 0.f};
  int L = 0;
  if (active && !PACKED) {
    if (d.dhT) Dh = d.dhT[(long)b * n + j];
    if (d.dcT) Dc = d.dcT[(long)b * n + j];
    L = clamp_len(a.lens, b, T);
  }
  // What the gate gradients of a frame need: gates, the cell state entering it, dy.
  // The per-frame arrays are read through buffer descriptors that cover exactly one frame: the frame's address is
  // scalar arithmetic, a lane's offset inside the frame never changes, and a lane with nothing to fetch (row past the
  // batch, unit past n, frame past the row's length) has its offset parked outside the frame and gets zeros without
  // touching memory - as does every lane when the frame itself does not exist (zero-sized descriptor).  Nothing is
  // predicated.  They come from HBM, and a compute unit hands loads back in the order of issue: the ring loads behind them wait.
  // Six loads a step cost 0.17 us of it; so a lane brings four units of a gate, the loads write LDS, three a frame, and kAhead frames
  // are fetched together (see the forward kernel; n = 1024: 2 frames 1.34 us a step, 4 1.33; 256 units: 0.99, 0.97).
  constexpr unsigned kParked = 0x7ff00000u;
  const unsigned g_bytes = (unsigned)B * 4u * n * 4u, s_bytes = (unsigned)B * n * 4u, y_bytes = (unsigned)B * d.lddy * 2u;
  const unsigned g_off = active ? ((unsigned)b * 4u * n + j) * 4u : kParked;
  const unsigned s_off = active ? ((unsigned)b * n + j) * 4u : kParked;
  const unsigned y_off = active ? ((unsigned)b * d.lddy + j) * 2u : kParked;
  // (a frame that does not exist: the lanes that would read it are parked, whatever the address)
  auto frame_of = [&](const void* base, int t, unsigned bytes) {
    if constexpr (PACKED) return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes * (unsigned)T, kBufFlags);      // (see the forward kernel)
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (long long)t * bytes), 0, bytes, kBufFlags);
  };
  const int zq = (lane >> 3) & 3, zu = J * 32 + 4 * (lane & 7);
  const int L_row = b < B && zu < n ? clamp_len(a.lens, b, T) : 0;
  const unsigned gq_off = ((unsigned)b * 4u * n + (unsigned)zq * n + zu) * 4u;
  auto lds_addr = [](const void* p) { return __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) const char*)p); };
  const unsigned lds_g = lds_addr(&in_g[0][wave][0][0][0]), lds_c = lds_addr(&in_c[0][wave][0]), lds_y = lds_addr(&in_y[0][wave][0]), lds_n = lds_addr(&in_n[0][wave][0]);
  // Frames of backward steps sigma, sigma + 1, ... (sigma = T-1-tau) into places sigma % (2 kAhead), ...; t < 0 and t >= L as one
  // comparison.  The cell state entering frame t is the state leaving the frame before it in processing order, which is the NEXT
  // backward step's frame: that step takes its c_new from here instead of loading it again.  So the value is also fetched where
  // frame t itself is padding but the frame before it is real (direction +1, t = the row's length).  The state entering the first
  // frame is the caller's and kept in a register.
  const int t_first = d.rev ? 0 : T - 1, dt = d.rev ? 1 : -1;          // frame of backward step sigma: t_first + dt * sigma
  const unsigned L_prev = (unsigned)(d.rev ? min(L, T - 1) : L);
  // (assembly: the compiler makes every later LDS read wait for all loads of this kind that it knows to be in flight)
  const unsigned before_off = (unsigned)dt * s_bytes;      // from a frame's cell state to that of the frame before it
  unsigned e_ahead[kAhead] = {};                           // table words of the frames that are fetched next
  auto look_ahead = [&](int sigma, int now) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < kAhead; ++f) e_ahead[f] = tab.at(sigma + f, now);
  };
  auto fetch_in = [&](int sigma) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < kAhead; ++f) {
      const unsigned place = (unsigned)(sigma + f) & (2 * kAhead - 1);
      if constexpr (PACKED) {
        const unsigned e = e_ahead[f];
        const bool on = (e & kRowValid) != 0u, before = on && !(e & kRowLast), first = on && (e & kRowFirst) != 0u;
        const unsigned so = frame_off(e, 4u * n) + 4u * j;
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(lds_g + place * (unsigned)sizeof(in_g[0])), "v"(on && zu < n ? frame_off(e, 16u * n) + ((unsigned)zq * n + zu) * 4u : kParked), "s"(frame_of(d.gates, 0, g_bytes)) : "memory");
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(lds_c + place * (unsigned)sizeof(in_c[0])), "v"(before && active ? so + before_off : kParked), "s"(frame_of(d.cs, 0, s_bytes)) : "memory");
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(lds_n + place * (unsigned)sizeof(in_n[0])), "v"(first && active ? so : kParked), "s"(frame_of(d.cs, 0, s_bytes)) : "memory");
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_ushort %1, %2, 0 offen nt lds" ::"s"(lds_y + place * (unsigned)sizeof(in_y[0])), "v"(on && active ? frame_off(e, 2u * (unsigned)d.lddy) + 2u * j : kParked), "s"(frame_of(d.dy, 0, y_bytes)) : "memory");
        continue;
      }
      const int t = t_first + dt * (sigma + f), tp = t + dt;
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(lds_g + place * (unsigned)sizeof(in_g[0])), "v"((unsigned)t < (unsigned)L_row ? gq_off : kParked), "s"(frame_of(d.gates, t, g_bytes)) : "memory");
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(lds_c + place * (unsigned)sizeof(in_c[0])), "v"((unsigned)(d.rev ? t : tp) < L_prev ? s_off : kParked), "s"(frame_of(d.cs, tp, s_bytes)) : "memory");
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_ushort %1, %2, 0 offen nt lds" ::"s"(lds_y + place * (unsigned)sizeof(in_y[0])), "v"((unsigned)t < (unsigned)L ? y_off : kParked), "s"(frame_of(d.dy, t, y_bytes)) : "memory");
    }
  };
  tab.load(0);
  look_ahead(0, 0);
  fetch_in(0);
  const float c_first = !PACKED && active && d.c0 ? d.c0[(long)b * n + j] : 0.f;
  // cell state leaving the next step's frame: of the first one loaded as such
  float c_new = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.cs, t_first, s_bytes), t_first < L ? s_off : kParked, 0u, 2));
  // entries of DZ, which this thread stores: a pointer that moves by one frame per step
  const long row_last = (long)(d.rev ? 0 : T - 1) * B + b, g_step = (d.rev ? (long)B : -(long)B) * 4 * n;
  unsigned short* dz_p = (unsigned short*)d.DZ + row_last * 4 * n + j;

  // consumer side: a load covers two producers' blocks; lane reads output lane%32, all eight rows, of producer lane/32
  const int ccol = lane & 31, chalf = lane >> 5;
  const int nitv = (ntile2 + 7) / 8, rot = J % nitv;
  // (row group's part of the ring in bytes, below 2^31; wave-uniform by decree, see wg_coord)
  const unsigned ring_group = __builtin_amdgcn_readfirstlane((unsigned)R * ntile2 * ntile2 * kPartBytes), ring_tile = __builtin_amdgcn_readfirstlane(ring_group + (unsigned)(J * ntile2 * kPartBytes));
  // producer side: of a destination tile's two column tiles, lanes 0..31 publish the first and lanes 32..63 the second; a lane
  // rows 4*(lane/16 % 2) .. +3 of output column lane%16 + 16*(lane/32)
  const int pg = (lane >> 4) & 1, pcol = (lane >> 5) * 16 + (lane & 15);
  const int local = group_is_xcd_local(a.xcc, wg.base, ntile2, a.spin_limit);
  // byte offset, from row group R's part of the ring, of what this lane stores for destination tile wave*(NCT/2) + P (one past the
  // last falls outside the buffer): this producer's block, output column, row half
  unsigned pub_off[NCT / 2];
#pragma unroll
  for (int P = 0; P < NCT / 2; ++P) pub_off[P] = (unsigned)((((wave * (NCT / 2) + P) * ntile2 + J) * 32 + pcol) * 2 + pg) * 8u;

  PROF_DECL
  // One time step.
  // `ring_c`: the step reads partial sums (every step but the first); `pointwise_c`: it has a frame (every step but the
  // last, which only collects the Dh that leaves the layer).  Constants of the call, so that the loop below is free
  // of the two exceptions: with them inside, the compiler's wait counts in the loop allowed for paths it never takes.
  // `local_c`: the cache policy of the publishing stores.
  auto step = [&](const int tau, auto local_c, auto ring_c, auto pointwise_c) __attribute__((always_inline)) {
    PROF_MARK(4)
    // (told to be wave-uniform: computed next to per-lane uses of tau it ends up in vector registers, and a buffer
    // descriptor derived from it is then applied lane by lane in a loop)
    const int sigma = __builtin_amdgcn_readfirstlane(Tn - 1 - tau);
    const unsigned e = pointwise_c ? tab.at(sigma, sigma) : 0u;
    const int t = d.rev ? T - 1 - tau : tau;
    const int t_next = d.rev ? t - 1 : t + 1;
    constexpr bool pointwise = decltype(pointwise_c)::value;
    const bool valid = pointwise && active && (PACKED ? (e & kRowValid) != 0u : t < L);

    // The gate gradients of a valid frame, dh = dy + Dh (recurrent_dev.h has the plain form):
    //   dc = Dc + dh go (1 - tanh(c)^2), Dc' = dc gf, dz = (dc gg gi (1-gi), dc c_prev gf (1-gf), dc gi (1-gg^2), dh tanh(c) go (1-go)).
    // Everything that does not involve dh or Dc is computed while the ring loads are in flight.
    struct { float gi, gf, gg, go, c_new, c_prev; unsigned dy_bits; } in;
    auto take_in = [&]() __attribute__((always_inline)) {
      const int place = sigma & (2 * kAhead - 1);
      asm volatile("" ::: "memory");
      in.gi = in_g[place][wave][lane >> 5][0][u]; in.gf = in_g[place][wave][lane >> 5][1][u];
      in.gg = in_g[place][wave][lane >> 5][2][u]; in.go = in_g[place][wave][lane >> 5][3][u];
      in.c_new = c_new; in.c_prev = in_c[place][wave][lane]; in.dy_bits = in_y[place][wave][lane];
      if constexpr (PACKED) {
        if ((sigma & (kAhead - 1)) == 0) look_ahead(sigma + kAhead, sigma);
        if (e & kRowFirst) in.c_new = in_n[place][wave][lane];
        if ((e & kRowLast) && active && d.c0) in.c_prev = rare_load(&d.c0[(long)((e & kRowFrame) % (unsigned)B) * n + j]);
      } else if (tau == 0) {
        in.c_prev = c_first;
      }
      c_new = in.c_prev;
    };
    // Frames are asked for a step earlier than they could be: what a step computes from its inputs alone then runs while its poll is
    // in flight.
    auto fetch_next = [&]() __attribute__((always_inline)) {
      if ((sigma & (kAhead - 1)) == 0) fetch_in(sigma + kAhead);
    };
    float f_c = 0.f, f_i = 0.f, f_f = 0.f, f_g = 0.f, f_o = 0.f;
    auto factors = [&]() __attribute__((always_inline)) {
      if (valid) {
        const float tc = tanhf_(in.c_new);
        f_c = in.go * (1.f - tc * tc);
        f_i = in.gg * in.gi * (1.f - in.gi);
        f_f = in.c_prev * in.gf * (1.f - in.gf);
        f_g = in.gi * (1.f - in.gg * in.gg);
        f_o = tc * in.go * (1.f - in.go);
      }
    };
    // Accumulators, cleared while the ring loads are in flight (behind an assembly statement, or the compiler clears them where
    // they are used, in the way of what publishes).
    f32x4 acc[NCT / 2];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int P = 0; P < NCT / 2; ++P) acc[P] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int P = 0; P < NCT / 2; ++P) asm volatile("" : "+v"(acc[P]));
    };
    if constexpr (decltype(ring_c)::value) {
      RingReader rd;
      rd.rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)(((sigma - 1) & 1) ? d.ring1 : d.ring0) + ring_tile), 0, __builtin_amdgcn_readfirstlane(ntile2 * kPartBytes),
                                                kBufFlags);
      // load `it` of this wavefront covers producers 2 * (wave + 4 * it) and the one after it (1 KiB)
      rd.voff = (unsigned)(wave * 2 * kPartBytes + lane * 16);
      rd.it_bytes = 8u * kPartBytes;
      rd.lim = ntile2 - 2 * wave - chalf; rd.lim_step = 8;
      rd.tag = part_tag(sigma) << 14; rd.err = err; rd.limit = a.spin_limit;
      rd.nitv = nitv; rd.rot = rot;
      constexpr int NLD = NPW / 2;                          // loads per wavefront
      float ps[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      {
        // The sums need no masking but the tag bit's: the shifts drop the other halves.  With one wavefront per SIMD what
        // bounds this phase is its instruction stream, and a verdict per load (compare, branch, or worse a ballot
        // handed to scalar registers) costs as much as the additions themselves.  So the loads behind the poll are
        // taken together: their values are added into sums of their own without looking, the tag differences are ORed
        // per lane, and one compare and branch decides whether those sums count.  If not, the loads are fetched
        // again, all at once, by fix_up_batch.
        auto add = [&](float (&acc)[8], const u32x4& v) __attribute__((always_inline)) {
          acc[0] += __uint_as_float(v[0] << 16); acc[1] += __uint_as_float(v[0] & 0xffff0000u);
          acc[2] += __uint_as_float(v[1] << 16); acc[3] += __uint_as_float(v[1] & (0xffff0000u & ~kLLFwdTagBit));
          acc[4] += __uint_as_float(v[2] << 16); acc[5] += __uint_as_float(v[2] & 0xffff0000u);
          acc[6] += __uint_as_float(v[3] << 16); acc[7] += __uint_as_float(v[3] & (0xffff0000u & ~kLLFwdTagBit));
        };
        static_assert(NLD >= 2, "the poll is two loads");
        u32x4 x[NLD];
        const unsigned tagw = rd.tag << 16;
        // The poll is the first two loads, repeated (bounded) until their tags have turned and then kept; the others
        // are issued behind it (see the forward kernel).
        auto poll_loads = [&]() __attribute__((always_inline)) {
          x[0] = rd.load_it(rd.it_of(0));
          x[1] = rd.load_it(rd.it_of(1));
        };
        auto polled_stale = [&]() __attribute__((always_inline)) {
          const unsigned stale = rd.tag_diff(x[0], rd.it_of(0), tagw) | rd.tag_diff(x[1], rd.it_of(1), tagw);
          return __builtin_amdgcn_ballot_w64(stale > 0xffffu) != 0ull;
        };
        poll_loads();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (pointwise) {                         // while the poll is in flight: all that does not need Dh
          take_in();
          clear();
          factors();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(polled_stale() && !dead, 0)) rd.poll_again(dead, poll_loads, polled_stale);
        PROF_MARK(5)
        // (nothing is in flight behind the poll, the next step's inputs included)
        __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0)
#pragma unroll
        for (int i = 2; i < NLD; ++i) x[i] = rd.load_it(rd.it_of(i));
        __builtin_amdgcn_sched_barrier(0);
        // while those loads are on their way: the polled loads' values
        add(ps, x[0]);
        add(ps, x[1]);
        __builtin_amdgcn_sched_barrier(0);
        unsigned long long redo = 0ull;
        if (NLD > 2) {
          float pg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          unsigned bad = 0u;
#pragma unroll
          for (int i = 2; i < NLD; ++i) {
            __builtin_amdgcn_sched_barrier(0);             // each load is waited for and consumed in turn
            bad |= rd.tag_diff(x[i], rd.it_of(i), tagw);
            add(pg, x[i]);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad > 0xffffu) == 0ull, 1)) {
#pragma unroll
            for (int v = 0; v < 8; ++v) ps[v] += pg[v];
          } else {
            redo |= ((1ull << NLD) - 1ull) & ~3ull;
          }
        }
        PROF_REDO(__popcll(redo))
        if (redo) {
          rd.fix_up_batch<NLD>(redo, dead, [&](int, const u32x4& v) __attribute__((always_inline)) { add(ps, v); });
          // (nothing of that is outstanding any more - said with an instruction the compiler takes note of: it cannot tell
          // from the loop's exits, and would make whatever reuses those registers below wait for every load in flight)
          __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0)
        }
        // The next frames' inputs, from HBM.  Loads complete in the order of issue: asked for in front of the groups
        // above (where their latency would be covered best) they held up every ring load behind them - a tenth of the step.
        if constexpr (pointwise) fetch_next();
      }
      PROF_MARK(0)
#pragma unroll
      for (int v = 0; v < 8; ++v) red[2 * wave + chalf][v][ccol] = ps[v];
      __syncthreads();
      if (active && (PACKED || t_next < L)) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += red[k][r8][u];
        Dh = sum * (1.f / kPartScale);                     // the partial sums travel scaled (see above)
        if constexpr (PACKED) {
          if ((e_prev & kRowLast) && (d.dh0 || d.dc0)) {   // the gradients that leave the row that ended
            const long s0 = (long)((e_prev & kRowFrame) % (unsigned)B) * n + j;
            if (d.dh0) d.dh0[s0] = Dh;
            if (d.dc0) d.dc0[s0] = Dc;
          }
        }
      }
    } else {
      __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
      take_in();
      clear();
      factors();
      fetch_next();
    }
    if (pointwise) {
      if constexpr (PACKED) {
        if ((e & kRowFirst) && active) {
          Dh = 0.f; Dc = 0.f;
          if (d.dhT || d.dcT) {
            const long s0 = (long)((e & kRowFrame) % (unsigned)B) * n + j;
            if (d.dhT) Dh = rare_load(&d.dhT[s0]);
            if (d.dcT) Dc = rare_load(&d.dcT[s0]);
          }
        }
        e_prev = e;
      }
      float dz[4] = {0.f, 0.f, 0.f, 0.f};
      if (valid) {
        const float dh = bf_bits2f((unsigned short)in.dy_bits) + Dh, dc = Dc + dh * f_c;
        Dc = dc * in.gf;
        dz[0] = dc * f_i; dz[1] = dc * f_f; dz[2] = dc * f_g; dz[3] = dh * f_o;
      }
      const unsigned b01 = pack_bf16x2(dz[0], dz[1]), b23 = pack_bf16x2(dz[2], dz[3]);
      const unsigned short bits[4] = {(unsigned short)b01, (unsigned short)(b01 >> 16), (unsigned short)b23, (unsigned short)(b23 >> 16)};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        dbsum[q] += dz[q];
        zb[r8][q * 32 + u] = bits[q];                      // inactive threads contribute zeros
      }
      __syncthreads();
      PROF_MARK(2)
      // Partial sums of Dh for all n outputs: [8 rows, K = 128] x [128, 256 outputs of this wave], four products for a destination
      // tile's two column tiles (see smfmac_b_agpr), published by ONE store of 8 bytes a lane.
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          (void*)((const char*)((sigma & 1) ? d.ring1 : d.ring0) + ring_group), 0, __builtin_amdgcn_readfirstlane(ntile2 * ntile2 * kPartBytes), kBufFlags);
      const unsigned tag_hi = part_tag(sigma + 1) << 30;
      u32x4 av[4];
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) av[kc] = *(const u32x4*)&zb[lane & 7][kc * 32 + (lane >> 4) * 8];
      // A product issues every 16 cycles, of which the wavefront's issue slot is taken for 4 (see the forward kernel for the
      // measurements).  What publishes a tile is cut into single instructions that follow the products of the next tiles,
      // from two products behind its last one on (by then its results have been written: more than the wait states between the two).
      // Nothing is predicated.
      constexpr bool kLocal = decltype(local_c)::value;
      constexpr int kPubSteps = 4, kPubLag = 2, kMma = 2 * NCT, kOps = NCT / 2 * kPubSteps;
      u32x2 val[2];
      auto pub_step = [&](int o) __attribute__((always_inline)) {
        if (o < 0 || o >= kOps) return;
        const int P = o / kPubSteps, kk = o % kPubSteps;
        u32x2& v = val[P & 1];
        if (kk == 0) v[0] = pack_bf16x2(acc[P][0], acc[P][1]);
        else if (kk == 1) v[1] = pack_bf16x2(acc[P][2], acc[P][3]);
        else if (kk == 2) v[1] |= tag_hi;                  // (bit 14 of the fourth value is 0 below 2^33: see the format)
        else __builtin_amdgcn_raw_buffer_store_b64(v, ro, pub_off[P], 0, kLocal ? 0 : 16);   // 16: sc1, agent scope, written through
      };
      operands_settle(av[0], av[1], av[2], av[3]);
#pragma unroll
      for (int i = 0; i < kMma; ++i) {
        smfmac_b_agpr(acc[i >> 2], av[i & 3], w[i & 3][i >> 2], sparse);
        __builtin_amdgcn_sched_barrier(0);
        pub_step(i - 3 - kPubLag);                         // (product 4P + 3 is destination tile P's last)
        __builtin_amdgcn_sched_barrier(0);
      }
      mfma_settle(acc[NCT / 2 - 2], acc[NCT / 2 - 1]);
#pragma unroll
      for (int o = kMma - 3 - kPubLag; o < kOps; ++o) pub_step(o);
      PROF_MARK(1)
      if constexpr (PACKED) {
        const __amdgpu_buffer_rsrc_t rz = frame_of(d.DZ, 0, g_bytes / 2u);
        const unsigned zo = valid ? frame_off(e, 8u * n) + 2u * j : kParked;
#pragma unroll
        for (int q = 0; q < 4; ++q) __builtin_amdgcn_raw_buffer_store_b16(bits[q], rz, zo, (unsigned)q * 2u * n, 2);
      } else {
        if (active) {
#pragma unroll
          for (int q = 0; q < 4; ++q) st_stream(dz_p + q * n, bits[q]);
        }
        dz_p += g_step;
      }
      PROF_MARK(3)
    }
  };
  // The time loop, once for each cache policy: with a branch around the products of every step both sides' accumulators are
  // alive together, and the compiler copies one set in front of its products.
  // (tau is told to be wave-uniform: computed next to per-lane uses it ends up in vector registers)
  auto all_steps = [&](auto local_c) __attribute__((always_inline)) {
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (Tn > 0) {
      step(Tn - 1, local_c, no, yes);
      for (int tau = Tn - 2; tau >= 0; tau = __builtin_amdgcn_readfirstlane(tau) - 1) {
        if (PACKED && ((Tn - 1 - tau) & (kTabSteps - 1)) == 0) tab.load(Tn - 1 - tau);
        step(tau, local_c, yes, yes);
      }
      step(-1, local_c, yes, no);
    }
  };
  if (local) all_steps(std::true_type{});
  else all_steps(std::false_type{});
  PROF_DUMP("bwdp", T)
  if constexpr (PACKED) {
    if (wg.rt == 0 && active && (d.dh0 || d.dc0))          // rows without frames
      for (int bb = r8; bb < B; bb += 8)
        if (clamp_len(a.lens, bb, T) == 0) {
          const long s0 = (long)bb * n + j;
          if (d.dh0) d.dh0[s0] = d.dhT ? d.dhT[s0] : 0.f;
          if (d.dc0) d.dc0[s0] = d.dcT ? d.dcT[s0] : 0.f;
        }
  } else if (active) {
    if (d.dh0) d.dh0[(long)b * n + j] = Dh;
    if (d.dc0) d.dc0[(long)b * n + j] = Dc;
  }
  if (d.dbpart) {                       // bias gradient: sum this work-group's 8 rows, one slice per row group
    auto& dbred = lds.dbred;
#pragma unroll
    for (int q = 0; q < 4; ++q) dbred[r8][q * 32 + u] = dbsum[q];
    __syncthreads();
    if (tid < 128) {
      const int q = tid >> 5, uu = tid & 31, jj = J * 32 + uu;
      float sum = 0.f;
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) sum += dbred[rr][q * 32 + uu];
      if (jj < n) d.dbpart[(long)R * 4 * n + q * n + jj] = sum;
    }
  }
}

// The same kernel for work-groups of 16 rows (two per thread: rows r8 and r8 + 8 of the group), for batches that the
// 8-row form cannot hold in one launch.  The MFMAs and the publishing stores are the same instructions with all 64 lanes
// doing real work; a (producer, destination tile) block is 1 KiB -
// [32 outputs][4 row quarters] x 8 bytes -, a consumer's load covers one producer (lane = output lane/2, row half lane%2),
// so a wavefront reads eight loads per step instead of four, and the pointwise part runs twice.
struct Bwd16Lds {
  static constexpr int kAhead = 2;                       // frames whose inputs are fetched together (see the 8-row kernel)
  alignas(16) float red[4][16][33];                      // [wavefront][row][output]
  alignas(16) unsigned short zb[16][136];
  alignas(16) float in_g[2 * kAhead][2][4][2][4][32];    // [frame][row half][wavefront]...
  alignas(16) float in_c[2 * kAhead][2][4][64];
  alignas(16) unsigned in_y[2 * kAhead][2][4][64];
  float dbred[8][129];
};
template <int NPW, int NCT>                               // n <= 128 * NPW (producers per wavefront) and n <= 64 * NCT (its output column tiles)
__device__ __forceinline__ void bwd16_body(const PBwdArgs& a, const GridMap& map, Bwd16Lds& lds) {
  constexpr int kAhead = Bwd16Lds::kAhead;
  auto& red = lds.red;
  auto& zb = lds.zb;
  auto& in_g = lds.in_g;
  auto& in_c = lds.in_c;
  auto& in_y = lds.in_y;
  constexpr int kBlock = 2 * kPartBytes;                 // one (producer, destination tile)
  const WgCoord wg = wg_coord(map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const PBwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int J = wg.tile, R = a.rt0 + wg.rt, ntile2 = a.map.ntile;         // R: row group of 16 rows, counted over the whole batch
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int n = a.n, B = a.B, T = a.T;
  unsigned* err = a.sync;
  bool dead = false;

  u32x4 w[4][NCT];                                       // all 256 accumulation registers at NCT = 16
#pragma unroll
  for (int kc = 0; kc < 4; ++kc)
#pragma unroll
    for (int c = 0; c < NCT; ++c) w[kc][c] = load_to_agpr(&d.Wb[((((long)J * 4 + wave) * 4 + kc) * NCT + c) * 64 + lane]);
  agpr_loads_done();

  const int r8 = tid >> 5, u = tid & 31;                 // pointwise pairs of this thread: rows r8 and r8 + 8, unit u
  const int b0 = R * 16 + r8, j = J * 32 + u;
  bool active[2];
  float Dh[2], Dc[2];
  float dbsum[4] = {0.f, 0.f, 0.f, 0.f};
  int L[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = b0 + 8 * k;
    active[k] = b < B && j < n;
    Dh[k] = 0.f; Dc[k] = 0.f; L[k] = 0;
    if (active[k]) {
      if (d.dhT) Dh[k] = d.dhT[(long)b * n + j];
      if (d.dcT) Dc[k] = d.dcT[(long)b * n + j];
      L[k] = clamp_len(a.lens, b, T);
    }
  }
  // What the gate gradients of a frame need, and how it is fetched: see the 8-row kernel.
  constexpr unsigned kParked = 0x7ff00000u;
  const unsigned g_bytes = in_sgpr((unsigned)B * 4u * n * 4u), s_bytes = in_sgpr((unsigned)B * n * 4u), y_bytes = in_sgpr((unsigned)B * d.lddy * 2u);
  // offsets of row r8 inside a frame; row r8 + 8 lies a wave-uniform distance behind it (and exists only if row r8 does)
  const unsigned g_off0 = active[0] ? ((unsigned)b0 * 4u * n + j) * 4u : kParked;
  const unsigned s_off0 = active[0] ? ((unsigned)b0 * n + j) * 4u : kParked;
  const unsigned y_off0 = active[0] ? ((unsigned)b0 * d.lddy + j) * 2u : kParked;
  auto g_off = [&](int k) { return k == 0 ? g_off0 : (active[1] ? g_off0 + 8u * 4u * n * 4u : kParked); };
  auto s_off = [&](int k) { return k == 0 ? s_off0 : (active[1] ? s_off0 + 8u * n * 4u : kParked); };
  auto y_off = [&](int k) { return k == 0 ? y_off0 : (active[1] ? y_off0 + 8u * (unsigned)d.lddy * 2u : kParked); };
  auto frame_of = [&](const void* base, int t, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + (long long)t * bytes), 0, bytes, kBufFlags);
  };
  const int zu = J * 32 + 4 * (lane & 7);
  int L_row[2];
  unsigned L_prev[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    L_row[k] = b0 + 8 * k < B && zu < n ? clamp_len(a.lens, b0 + 8 * k, T) : 0;
    L_prev[k] = (unsigned)(d.rev ? min(L[k], T - 1) : L[k]);
  }
  const unsigned gq_off = ((unsigned)b0 * 4u * n + ((unsigned)lane >> 3 & 3u) * n + zu) * 4u;
  auto lds_addr = [](const void* p) { return __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) const char*)p); };
  const unsigned lds_g = lds_addr(&in_g[0][0][wave][0][0][0]), lds_c = lds_addr(&in_c[0][0][wave][0]), lds_y = lds_addr(&in_y[0][0][wave][0]);
  const int t_first = d.rev ? 0 : T - 1, dt = d.rev ? 1 : -1;          // frame of backward step sigma: t_first + dt * sigma
  // (assembly: the compiler makes every later LDS read wait for all loads of this kind that it knows to be in flight)
  auto fetch_in = [&](int sigma) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < kAhead; ++f) {
      const unsigned place = (unsigned)(sigma + f) & (2 * kAhead - 1);
      const int t = t_first + dt * (sigma + f), tp = t + dt;
      const __amdgpu_buffer_rsrc_t rg = frame_of(d.gates, t, g_bytes), rc = frame_of(d.cs, tp, s_bytes), ry = frame_of(d.dy, t, y_bytes);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds_g + place * (unsigned)sizeof(in_g[0]) + (unsigned)(k * sizeof(in_g[0][0]))),
                     "v"((unsigned)t < (unsigned)L_row[k] ? gq_off : kParked), "s"(rg), "s"((unsigned)k * 8u * 4u * n * 4u) : "memory");
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(lds_c + place * (unsigned)sizeof(in_c[0]) + (unsigned)(k * sizeof(in_c[0][0]))),
                     "v"((unsigned)(d.rev ? t : tp) < L_prev[k] ? s_off(k) : kParked), "s"(rc) : "memory");
        asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_ushort %1, %2, 0 offen nt lds" ::"s"(lds_y + place * (unsigned)sizeof(in_y[0]) + (unsigned)(k * sizeof(in_y[0][0]))),
                     "v"((unsigned)t < (unsigned)L[k] ? y_off(k) : kParked), "s"(ry) : "memory");
      }
    }
  };
  fetch_in(0);
  float c_first[2], c_new[2];                              // cell state entering the first frame; leaving the next step's frame
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    c_first[k] = active[k] && d.c0 ? d.c0[(long)(b0 + 8 * k) * n + j] : 0.f;
    c_new[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(frame_of(d.cs, t_first, s_bytes), t_first < L[k] ? s_off(k) : kParked, 0u, 2));
  }
  // entries of DZ, which this thread stores: a pointer that moves by one frame per step
  const long row_last = (long)(d.rev ? 0 : T - 1) * B + b0, g_step = (d.rev ? (long)B : -(long)B) * 4 * n;
  unsigned short* dz_p = (unsigned short*)d.DZ + row_last * 4 * n + j;

  // consumer side: a load covers one producer's block; lane reads output lane/2, rows 8 * (lane%2) .. + 7
  const int ccol = lane >> 1, chalf = lane & 1;
  const int nitv = (ntile2 + 3) / 4, rot = J % nitv;
  // (row group's part of the ring in bytes, below 2^31; wave-uniform by decree, see wg_coord)
  const unsigned ring_group = __builtin_amdgcn_readfirstlane((unsigned)R * ntile2 * ntile2 * kBlock), ring_tile = __builtin_amdgcn_readfirstlane(ring_group + (unsigned)(J * ntile2 * kBlock));
  // producer side: lane holds rows 4*(lane/16) .. +3 of output column lane%16 of each accumulator tile
  const int pq = lane >> 4, pcol = lane & 15;
  const int local = group_is_xcd_local(a.xcc, wg.base, ntile2, a.spin_limit);
  // byte offset, from row group R's part of the ring, of what this lane stores for accumulator tile c: destination tile
  // wave*8 + c/2 (one past the last falls outside the buffer), this producer's block, output column, row quarter
  unsigned pub_off[NCT];
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    const int Jd = wave * (NCT / 2) + (c >> 1);
    pub_off[c] = (unsigned)(((Jd * ntile2 + J) * 32 + (c & 1) * 16 + pcol) * 4 + pq) * 8u;
  }

  PROF_DECL
  // One time step.
  // `ring_c`: the step reads partial sums (every step but the first); `pointwise_c`: it has a frame (every step but the
  // last, which only collects the Dh that leaves the layer).  Constants of the call, so that the loop below is free
  // of the two exceptions: with them inside, the compiler's wait counts in the loop allowed for paths it never takes.
  auto step = [&](const int tau, auto ring_c, auto pointwise_c) __attribute__((always_inline)) {
    PROF_MARK(4)
    // (told to be wave-uniform: computed next to per-lane uses of tau it ends up in vector registers, and a buffer
    // descriptor derived from it is then applied lane by lane in a loop)
    const int sigma = __builtin_amdgcn_readfirstlane(T - 1 - tau);
    const int t = d.rev ? T - 1 - tau : tau;
    const int t_next = d.rev ? t - 1 : t + 1;
    constexpr bool pointwise = decltype(pointwise_c)::value;
    bool valid[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) valid[k] = pointwise && active[k] && t < L[k];

    // The gate gradients of a valid frame, dh = dy + Dh (recurrent_dev.h has the plain form):
    //   dc = Dc + dh go (1 - tanh(c)^2), Dc' = dc gf, dz = (dc gg gi (1-gi), dc c_prev gf (1-gf), dc gi (1-gg^2), dh tanh(c) go (1-go)).
    // Everything that does not involve dh or Dc is computed while the ring loads are in flight.
    struct { float gi, gf, gg, go, c_new, c_prev; unsigned dy_bits; } in[2];
    auto take_in = [&]() __attribute__((always_inline)) {
      const int place = sigma & (2 * kAhead - 1);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        in[k].gi = in_g[place][k][wave][lane >> 5][0][u]; in[k].gf = in_g[place][k][wave][lane >> 5][1][u];
        in[k].gg = in_g[place][k][wave][lane >> 5][2][u]; in[k].go = in_g[place][k][wave][lane >> 5][3][u];
        in[k].c_new = c_new[k]; in[k].c_prev = in_c[place][k][wave][lane]; in[k].dy_bits = in_y[place][k][wave][lane];
        if (tau == 0) in[k].c_prev = c_first[k];
        c_new[k] = in[k].c_prev;
      }
    };
    float f_c[2], f_i[2], f_f[2], f_g[2], f_o[2];
    auto factors = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        f_c[k] = 0.f; f_i[k] = 0.f; f_f[k] = 0.f; f_g[k] = 0.f; f_o[k] = 0.f;
        if (valid[k]) {
          const float tc = tanhf_(in[k].c_new);
          f_c[k] = in[k].go * (1.f - tc * tc);
          f_i[k] = in[k].gg * in[k].gi * (1.f - in[k].gi);
          f_f[k] = in[k].c_prev * in[k].gf * (1.f - in[k].gf);
          f_g[k] = in[k].gi * (1.f - in[k].gg * in[k].gg);
          f_o[k] = tc * in[k].go * (1.f - in[k].go);
        }
      }
    };
    auto fetch_next = [&]() __attribute__((always_inline)) {
      if ((sigma & (kAhead - 1)) == 0) fetch_in(sigma + kAhead);
    };
    if constexpr (decltype(ring_c)::value) {
      RingReader rd;
      rd.rs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)(((sigma - 1) & 1) ? d.ring1 : d.ring0) + ring_tile), 0, __builtin_amdgcn_readfirstlane(ntile2 * kBlock),
                                                kBufFlags);
      // load `it` of this wavefront covers producer wave + 4 * it (1 KiB)
      rd.voff = (unsigned)(wave * kBlock + lane * 16);
      rd.it_bytes = 4u * kBlock;
      rd.lim = ntile2 - wave; rd.lim_step = 4;
      rd.tag = part_tag(sigma) << 14; rd.err = err; rd.limit = a.spin_limit;
      rd.nitv = nitv; rd.rot = rot;
      constexpr int NLD = NPW;                              // loads per wavefront
      float ps[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      {
        // The sums need no masking but the tag bit's: the shifts drop the other halves.  With one wavefront per SIMD what
        // bounds this phase is its instruction stream, and a verdict per load (compare, branch, or worse a ballot
        // handed to scalar registers) costs as much as the additions themselves.  So the loads behind the poll are
        // taken together: their values are added into sums of their own without looking, the tag differences are ORed
        // per lane, and one compare and branch decides whether those sums count.  If not, the loads are fetched
        // again, all at once, by fix_up_batch.
        auto add = [&](float (&acc)[8], const u32x4& v) __attribute__((always_inline)) {
          acc[0] += __uint_as_float(v[0] << 16); acc[1] += __uint_as_float(v[0] & 0xffff0000u);
          acc[2] += __uint_as_float(v[1] << 16); acc[3] += __uint_as_float(v[1] & (0xffff0000u & ~kLLFwdTagBit));
          acc[4] += __uint_as_float(v[2] << 16); acc[5] += __uint_as_float(v[2] & 0xffff0000u);
          acc[6] += __uint_as_float(v[3] << 16); acc[7] += __uint_as_float(v[3] & (0xffff0000u & ~kLLFwdTagBit));
        };
        static_assert(NLD >= 2, "the poll is two loads");
        u32x4 x[NLD];
        const unsigned tagw = rd.tag << 16;
        // The poll is the first two loads, repeated (bounded) until their tags have turned and then kept; the others
        // are issued behind it (see the forward kernel).
        auto poll_loads = [&]() __attribute__((always_inline)) {
          x[0] = rd.load_it(rd.it_of(0));
          x[1] = rd.load_it(rd.it_of(1));
        };
        auto polled_stale = [&]() __attribute__((always_inline)) {
          const unsigned stale = rd.tag_diff(x[0], rd.it_of(0), tagw) | rd.tag_diff(x[1], rd.it_of(1), tagw);
          return __builtin_amdgcn_ballot_w64(stale > 0xffffu) != 0ull;
        };
        poll_loads();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (pointwise) {                         // while the poll is in flight: all that does not need Dh
          take_in();
          factors();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(polled_stale() && !dead, 0)) rd.poll_again(dead, poll_loads, polled_stale);
        PROF_MARK(5)
        // (nothing is in flight behind the poll, the next step's inputs included)
        __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0)
#pragma unroll
        for (int i = 2; i < NLD; ++i) x[i] = rd.load_it(rd.it_of(i));
        __builtin_amdgcn_sched_barrier(0);
        // while those loads are on their way: the polled loads' values
        add(ps, x[0]);
        add(ps, x[1]);
        __builtin_amdgcn_sched_barrier(0);
        unsigned long long redo = 0ull;
        constexpr int kGroup = (NLD - 2) / 2;              // the other loads: two groups
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int i0 = 2 + g * kGroup, i1 = g == 0 ? 2 + kGroup : NLD;
          float pg[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          unsigned bad = 0u;
#pragma unroll
          for (int i = i0; i < i1; ++i) {
            __builtin_amdgcn_sched_barrier(0);             // each load is waited for and consumed in turn
            bad |= rd.tag_diff(x[i], rd.it_of(i), tagw);
            add(pg, x[i]);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad > 0xffffu) == 0ull, 1)) {
#pragma unroll
            for (int v = 0; v < 8; ++v) ps[v] += pg[v];
          } else {
            redo |= ((1ull << i1) - 1ull) & ~((1ull << i0) - 1ull);
          }
        }
        PROF_REDO(__popcll(redo))
        if (redo) {
          rd.fix_up_batch<NLD>(redo, dead, [&](int, const u32x4& v) __attribute__((always_inline)) { add(ps, v); });
          // (nothing of that is outstanding any more - said with an instruction the compiler takes note of: it cannot tell
          // from the loop's exits, and would make whatever reuses those registers below wait for every load in flight)
          __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0)
        }
        // The next frame's inputs, from HBM.  Loads complete in the order of issue: asked for in front of the groups
        // above (where their latency would be covered best) they held up every ring load behind them - a tenth of the step.
        if constexpr (pointwise) fetch_next();
      }
      PROF_MARK(0)
#pragma unroll
      for (int v = 0; v < 8; ++v) red[wave][8 * chalf + v][ccol] = ps[v];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (active[k] && t_next < L[k]) {
          const int rr = r8 + 8 * k;
          Dh[k] = (red[0][rr][u] + red[1][rr][u] + red[2][rr][u] + red[3][rr][u]) * (1.f / kPartScale);   // the partial sums travel scaled
        }
    } else {
      __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
      take_in();
      factors();
      fetch_next();
    }
    if (pointwise) {
      unsigned short bits[2][4];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        float dz[4] = {0.f, 0.f, 0.f, 0.f};
        if (valid[k]) {
          const float dh = bf_bits2f((unsigned short)in[k].dy_bits) + Dh[k], dc = Dc[k] + dh * f_c[k];
          Dc[k] = dc * in[k].gf;
          dz[0] = dc * f_i[k]; dz[1] = dc * f_f[k]; dz[2] = dc * f_g[k]; dz[3] = dh * f_o[k];
        }
        const unsigned b01 = pack_bf16x2(dz[0], dz[1]), b23 = pack_bf16x2(dz[2], dz[3]);
        bits[k][0] = (unsigned short)b01; bits[k][1] = (unsigned short)(b01 >> 16);
        bits[k][2] = (unsigned short)b23; bits[k][3] = (unsigned short)(b23 >> 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          dbsum[q] += dz[q];
          zb[r8 + 8 * k][q * 32 + u] = bits[k][q];         // inactive threads contribute zeros
        }
      }
      __syncthreads();
      PROF_MARK(2)
      // partial sums of Dh for all n outputs: [16 rows, K = 128] x [128, 256 outputs of this wave],
      // in four groups of four column tiles: while the MFMAs of one group run, the previous group's results are
      // converted and stored.  One 16-byte store per accumulator tile: the 32 storing lanes of a wavefront cover 512
      // consecutive bytes.  Each 8-byte half carries its own tag in its upper dword, so the only thing relied on
      // beyond the 64-bit units of the other kernels is that an aligned 16-byte lane store is not split below 8 bytes.
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          (void*)((const char*)((sigma & 1) ? d.ring1 : d.ring0) + ring_group), 0, __builtin_amdgcn_readfirstlane(ntile2 * ntile2 * kBlock), kBufFlags);
      const unsigned tag_hi = part_tag(sigma + 1) << 30;
      u32x4 av[4];
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) av[kc] = *(const u32x4*)&zb[lane & 15][kc * 32 + (lane >> 4) * 8];
      f32x4 acc[NCT];
      // NCT column tiles, the k loop inside.  An MFMA of this shape issues every 16 cycles, of which the wavefront's
      // issue slot is taken for 4 (see the forward kernel for the measurements).  What publishes a tile (two conversions,
      // three moves and one store) is cut into single instructions that follow the MFMAs of the tile two behind it:
      // by then its last result has been written (more than the 20 wait states mfma_settle would spend), the
      // instructions cost little there, and only the last two tiles are published behind the last MFMA (with groups of
      // four tiles, as this was first written, a whole group's publishing - a quarter of it - trailed the stream).
      // Nothing is predicated: lanes that hold no result have their store offset parked outside the buffer (pub_off),
      // and the two cache policies are two copies of the code.
      constexpr int kPubSteps = 4, kPubLag = 2;             // a tile is published behind the MFMAs of the tile kPubLag after it
      auto mma_publish = [&](auto local_c) __attribute__((always_inline)) {
        constexpr bool kLocal = decltype(local_c)::value;
        u32x2 val[4];
        auto pub_step = [&](int c, int kk) __attribute__((always_inline)) {
          u32x2& v = val[c & 3];
          if (kk == 0) v[0] = pack_bf16x2(acc[c][0], acc[c][1]);
          else if (kk == 1) v[1] = pack_bf16x2(acc[c][2], acc[c][3]);
          else if (kk == 2) v[1] |= tag_hi;                  // (bit 14 of the fourth value is 0 below 2^33: see the format)
          else __builtin_amdgcn_raw_buffer_store_b64(v, ro, pub_off[c], 0, kLocal ? 0 : 16);   // 16: sc1, agent scope, written through
        };
        operands_settle(av[0], av[1], av[2], av[3]);
#pragma unroll
        for (int c = 0; c < NCT; ++c)
#pragma unroll
          for (int kc = 0; kc < 4; ++kc) {
            if (kc == 0) mfma_b_agpr_first(acc[c], av[kc], w[kc][c]);
            else mfma_b_agpr(acc[c], av[kc], w[kc][c]);
            if (c >= kPubLag) {                              // one step of the earlier tile behind each MFMA
              __builtin_amdgcn_sched_barrier(0);
              pub_step(c - kPubLag, kc);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        mfma_settle(acc[NCT - 4], acc[NCT - 3], acc[NCT - 2], acc[NCT - 1]);
#pragma unroll
        for (int c = NCT - kPubLag; c < NCT; ++c)
#pragma unroll
          for (int k = 0; k < kPubSteps; ++k) pub_step(c, k);
      };
      // (opaque in every step: the compiler would make two copies of the whole time loop otherwise)
      int local_ = local;
      asm volatile("" : "+s"(local_));
      if (local_) mma_publish(std::true_type{});
      else mma_publish(std::false_type{});
      PROF_MARK(1)
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (active[k]) {
#pragma unroll
          for (int q = 0; q < 4; ++q) st_stream(dz_p + (long)k * 8 * 4 * n + q * n, bits[k][q]);
        }
      dz_p += g_step;
      PROF_MARK(3)
    }
  };
  // (tau is told to be wave-uniform: computed next to per-lane uses it ends up in vector registers)
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  step(T - 1, no, yes);                                    // (T >= 2)
  for (int tau = T - 2; tau >= 0; tau = __builtin_amdgcn_readfirstlane(tau) - 1) step(tau, yes, yes);
  step(-1, yes, no);
  PROF_DUMP("bwdp16", T)
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (active[k]) {
      if (d.dh0) d.dh0[(long)(b0 + 8 * k) * n + j] = Dh[k];
      if (d.dc0) d.dc0[(long)(b0 + 8 * k) * n + j] = Dc[k];
    }
  if (d.dbpart) {                       // bias gradient: sum this work-group's 16 rows into the first of its two slices (the other stays zero)
    auto& dbred = lds.dbred;
#pragma unroll
    for (int q = 0; q < 4; ++q) dbred[r8][q * 32 + u] = dbsum[q];
    __syncthreads();
    if (tid < 128) {
      const int q = tid >> 5, uu = tid & 31, jj = J * 32 + uu;
      float sum = 0.f;
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) sum += dbred[rr][q * 32 + uu];
      if (jj < n) d.dbpart[(long)2 * R * 4 * n + q * n + jj] = sum;
    }
  }
}

// The kernels.  Fewer rows than a launch holds: every row has a place of its own (8 rows a group).  More: 16 rows a group, or, for n
// where the choice below is offered, rows one behind the other in the places of the 8-row form.
template <int NL>
__global__ __launch_bounds__(256) void persist_fwd8_kernel(PFwdArgs a) {
  __shared__ Fwd8Lds<false, false> lds;
  fwd8_body<NL, false>(a, lds);
}
template <int NL>
__global__ __launch_bounds__(256) void persist_fwd8_rows_w_kernel(PFwdArgs a) {
  __shared__ Fwd8Lds<false, true> lds;
  fwd8_body<NL, false, true>(a, lds);
}
template <int NIT>
__global__ __launch_bounds__(256) void persist_fwd16r_kernel(PFwdArgs a) {
  __shared__ Fwd16Lds<NIT> lds;
  fwd16_body<NIT>(a, a.map, lds);
}
template <int NPW, int NCT>
__global__ __launch_bounds__(256) void persist_bwdp_kernel(PBwdArgs a) {
  __shared__ Bwd8Lds<NCT, false> lds;
  bwd8_body<NPW, NCT, false>(a, lds);
}
template <int NPW, int NCT>
__global__ __launch_bounds__(256) void persist_bwdp16_kernel(PBwdArgs a) {
  __shared__ Bwd16Lds lds;
  bwd16_body<NPW, NCT>(a, a.map, lds);
}
__device__ __forceinline__ GridMap rows16_map(GridMap m, int B) {
  m.nrow = (B + 15) / 16;                                  // (no more groups than the grid is for: persist_pack_slots)
  return m;
}
// The lengths decide (rows_pay), and they are on the device: the set-up launch writes the decision with the table.
__global__ __launch_bounds__(256) void persist_fwd_rows_kernel(PFwdArgs a) {
  __shared__ union { Fwd8Lds<true, false> r8; Fwd16Lds<8> r16; } lds;
  if (__builtin_amdgcn_readfirstlane(a.steps[0]) >= 0) fwd8_body<4, true>(a, lds.r8);
  else fwd16_body<8>(a, rows16_map(a.map, a.B), lds.r16);
}
__global__ __launch_bounds__(256) void persist_bwd_rows_kernel(PBwdArgs a) {
  __shared__ union { Bwd8Lds<16, true> r8; Bwd16Lds r16; } lds;
  if (__builtin_amdgcn_readfirstlane(a.steps[0]) >= 0) bwd8_body<8, 16, true>(a, lds.r8);
  else bwd16_body<8, 16>(a, rows16_map(a.map, a.B), lds.r16);
}

// ------------------------------------------------------------------------------------------------
// forward, float storage.  The float MFMA (16x16x4) runs at a sixteenth of the bfloat16 rate, 7.1 us per step for 64 rows
// x 2 directions of n = 1000 on the whole device; so a product is six bfloat16 ones of three-part sums (Splitter: 24 bits, as float), 2.7 us, and
// errors against 64 bits are 0.6 of what float MFMAs gave (y 2.6e-7 -> 1.6e-7 of its size, dW_h 5.0e-7 -> 2.8e-7; n = 160 to 1000, weights up to 6 / sqrt n).  A step's tags
// are looked at before its products, all of them, and h is split between products of the pair before.  What bounds a step now is the exchange:
// us a step, forward and backward, 64 rows x 2 directions of n = 1024 12.0 and 14.3 -> 8.2 and 12.1, 16 rows 6.8 and 6.9 -> 4.2 and 5.5, of
// n = 512 4.4 and 4.4 -> 2.4 and 3.4, of 256 2.8 and 2.9 -> 1.85 and 2.4.
// Two things matter to it.  (1) Every work-group reads the whole h of its rows in float, from
// beyond L2 (an exchange group spans several XCDs), so rows per work-group are traded against copies of W_h: a work-group
// owns 16 units - 64 gate columns, four MFMA column tiles - for a slab of 32 rows: 63 x 2 slabs x 2 directions = 252
// work-groups for config 2, W_h held twice on the device (256 registers per lane: the per-step kernel's packed slices of
// two 8-unit tiles), 128 KiB of ring read per work-group and step (with 8 units x 64 rows, 256 KiB, a step of float MFMAs took 13.8 us
// against 11 for its products alone).  (2) The round trip of the exchange - reduce, cell, publish, and the consumers' loads,
// about 2.5 us - which nothing overlaps if all rows move in lock step (12.0 us per step).  The two row tiles of a slab
// are different batch rows, i.e. independent recurrences: they are walked HALF A STEP APART, one's products running
// while the other's h travels.
// The K axis is split over the four wavefronts (chunks of 16 k, wavefront w takes chunks w, w + 4, ...), their accumulators
// meet in LDS, a thread updates one cell per row tile, and two neighbouring units are published as ONE 8-byte unit of the
// ring: two float h values, the tag in bit 30 of the second (|h| <= 1 leaves the top exponent bit 0, as bit 14 of a
// bfloat16 value in the other kernels; a NaN there goes into the first).  The ring is the per-step kernel's fragment-ordered h buffer [row tile][chunk][lane]
// x 16 bytes, a lane's 16 bytes being two such units, so the reader of the other kernels applies unchanged.  An initial
// hidden state never enters the ring (it is not bounded by 1): rows publish zeros until their first frame is done, and
// h0 W_h has been added to that frame's pre-activations.
// Rows are dealt to row tiles by falling length, and a slab is a long tile together with a short one: a row tile leaves its
// loop (reversed: enters it) at its longest row's last frame - every work-group of the exchange group knows it from the lengths - and its
// half of every step beyond that costs nothing but the stores of padding.  (Config 2, rows of 10 - 50 frames in any order: the four tiles
// work 50, 40, 30 and 20 of 50 steps: forward 594 -> 470 us, backward 703 -> 538.)  Rows beyond 256 stay where they are.  With a single row tile per slab (whenever the device
// holds the launch that way) a step has no other half to wait for.
// order[slot] = row; called by all 256 threads
__device__ __forceinline__ void rows_by_length(int* order, int* len, const int* lens, int B, int T) {
  const int b = threadIdx.x;
  if (b < B) len[b] = clamp_len(lens, b, T);
  __syncthreads();
  if (b < B) {
    int rank = 0;
    for (int o = 0; o < B; ++o) rank += len[o] > len[b] || (len[o] == len[b] && o < b);
    order[rank] = b;
  }
  __syncthreads();
}
// What a work-group of the float kernels works on: row tiles (of rows in falling length), the rows of this thread's cells (pointwise row r16), and
// the steps that a tile takes part in, as positions in processing order [first, first + count).
struct F32Rows {
  int count_tiles, tile[2], row[2], first[2], count[2];      // row: -1 = none
};
__device__ __forceinline__ F32Rows f32_rows(const int* lens, int B, int T, bool rev, int slab, int slab_tiles, int r16) {
  __shared__ int order[256], len[256];
  const bool sorted = lens != nullptr && B <= 256;
  if (sorted) rows_by_length(order, len, lens, B, T);
  F32Rows f;
  const int nrt = (B + 15) / 16;
  f.tile[0] = slab; f.tile[1] = nrt - 1 - slab;
  f.count_tiles = slab_tiles == 2 && f.tile[1] > f.tile[0] ? 2 : 1;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int slot = f.tile[k] * 16 + r16;
    f.row[k] = k < f.count_tiles && slot < B ? (sorted ? order[slot] : slot) : -1;
    f.count[k] = __builtin_amdgcn_readfirstlane(sorted && k < f.count_tiles ? len[order[f.tile[k] * 16]] : T);    // (the tile's first row is its longest)
    f.first[k] = rev ? T - f.count[k] : 0;
  }
  return f;
}

// A float as the sum of three bfloat16 (8 + 8 + 8 bits, rounded to nearest, the last exactly; gemm_float.hip), eight of them in twelve small steps that
// fit between products: part e / 4 of elements 2 (e % 4) and the next.  Exactly from 2^-110 up: what may be smaller is scaled by a power of two first (W_h, and dz of the
// backward loop).  h is not: what its parts lose, 2^-134, times weights below 2^76 is below 2^-48 in a pre-activation, which gates that are good to 2^-24 cannot feel.
struct Splitter {
  float v[8];
  u32x4 part[3];
  __device__ __forceinline__ void step(int e) {
    float &lo = v[2 * (e & 3)], &hi = v[2 * (e & 3) + 1];
    const unsigned u = pack_bf16x2(lo, hi);
    part[e >> 2][e & 3] = u;
    if (e < 8) { lo -= __uint_as_float(u << 16); hi -= __uint_as_float(u & 0xffff0000u); }
  }
};
constexpr float kWScale = 0x1p40f;
constexpr float kBwdScale = 0x1p24f, kSumScale = kPartScale / (kBwdScale * kBwdScale);    // backward: of dz and of W_h^T; of their sums on their way
constexpr unsigned kWMost = 0x79800000u;                   // 2^116: a sum of 256 products with h stays finite
template <int NCH>                                         // chunks per wavefront at most: n <= 64 * NCH
__global__ __launch_bounds__(256) void persist_fwd_f32_kernel(PFwdArgs a) {
  constexpr int NP = NCH / 2;                              // pairs of chunks: 32 k, the depth of a bfloat16 product
  __shared__ float red[4][16][65];
  __shared__ u32x4 w_low[4][NP][4][64];                    // [wavefront][pair][column tile][lane]
  __shared__ float zxs[2][4][4][NCH <= 8 ? 64 : 1];        // [step][wavefront][gate][lane]
  const WgCoord wg = wg_coord(a.map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const int tile = wg.tile;                                // 16 units
  const PFwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkc = a.nkc, n = a.n, B = a.B, T = a.T;
  const int ntile8 = (n + 7) / 8;
  unsigned* err = a.sync;
  bool dead = false;

  // W_h slice: chunk kc = wave + 4 it; column tile ct = tile of 8 units (ct >> 1), its gates i,f (ct & 1 = 0) or g,o
  // (the per-step kernel's packing)
  // In three bfloat16 parts: two fill the 256 accumulation registers of every lane and the MFMAs read them there (inline assembly, as in the
  // bfloat16 kernels), the smallest lies in LDS, where a wavefront reads back what it wrote.  A chunk past the end of K or a column
  // tile past n takes the last valid one's weights instead of zeros: the h values of such a chunk arrive as zeros (the ring's descriptor ends before
  // them), and such columns are never stored.
  u32x4 wh[NP][4], wm[NP][4];
  unsigned w_most = 0u;
  auto w_at = [&](int it, int ct) __attribute__((always_inline)) {
    const int kc = min(wave + 4 * it, nkc - 1), tile8 = min(tile * 2 + (ct >> 1), ntile8 - 1);
    return *((const u32x4*)d.Wf + ((long)(tile8 * 2 + (ct & 1)) * nkc + kc) * 64 + lane);
  };
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    u32x4 v[4][2];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) { v[ct][0] = w_at(2 * p, ct); v[ct][1] = w_at(2 * p + 1, ct); }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      Splitter s;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        s.v[e] = __uint_as_float(v[ct][e >> 2][e & 3]) * kWScale;
        w_most = max(w_most, __float_as_uint(s.v[e]) & 0x7fffffffu);
      }
#pragma unroll
      for (int e = 0; e < 12; ++e) s.step(e);
      wh[p][ct] = s.part[0];
      wm[p][ct] = s.part[1];
      w_low[wave][p][ct][lane] = s.part[2];
      asm volatile("" : "+a"(wh[p][ct]), "+a"(wm[p][ct]));
    }
  }
  // Weights that the parts cannot hold (infinities, NaN, 2^76 and more): this wavefront's products are float MFMAs, W_h from memory.
  const bool plain = __builtin_amdgcn_ballot_w64(w_most >= kWMost) != 0ull;
  const int local = NCH <= 8 ? group_is_xcd_local(a.xcc, wg.base, a.map.ntile, a.spin_limit) : 0;      // (more than 32 members never are)

  const unsigned zxs_wave = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&zxs[0][wave][0][0]);
  // pointwise: row r16 of each row tile, unit u of the tile's 16
  const int r16 = tid >> 4, u = tid & 15;
  const int j = tile * 16 + u;
  const F32Rows rows = f32_rows(a.lens, B, T, d.rev, a.slab0 + wg.rt, a.slab_tiles, r16);
  const int nrt_here = rows.count_tiles;
  float c[2] = {0.f, 0.f}, h[2] = {0.f, 0.f};
  int L[2] = {0, 0};
  bool active[2];
  // A row publishes zeros until its first frame has been processed: its initial hidden state (not bounded by 1, so not
  // fit for the ring) reaches that frame through the pre-activations instead.
  bool started[2] = {false, false};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = rows.row[k];
    active[k] = b >= 0 && j < n;
    if (active[k]) {
      if (d.c0) c[k] = d.c0[(long)b * n + j];
      if (d.h0) h[k] = d.h0[(long)b * n + j];
      L[k] = clamp_len(a.lens, b, T);
    }
  }
  // The even unit of a pair publishes both: chunk j / 16, lane group (j % 16) / 4, half ((j % 4) / 2) of that lane's 16 bytes
  constexpr unsigned kParked = 0x7ff00000u;
  const bool publishes = (u & 1) == 0 && (j & ~3) < n;     // (readers look at whole quads of units: those past n are published as zeros)
  const unsigned pub_in_tile = (unsigned)((((long)(j >> 4) * 64 + ((j & 15) >> 2) * 16 + r16) * 2 + ((j >> 1) & 1)) * 8);
  const unsigned ring_bytes = (unsigned)((B + 15) / 16) * nkc * 1024u;
  const long fg = (long)B * 4 * n, fy = (long)B * d.ldy, fs = (long)B * n;     // elements per frame
  // columns of this thread's cell among the work-group's 64: 32 per tile of 8 units, then gate q, unit
  const int col0 = (u >> 3) * 32 + (u & 7);
  PROF_DECL
  // A half step's ring loads go out before the reduction and the cell update of the half step before it (their values were published half a
  // step earlier) and are there when the products begin.
  auto in_loop = [&](int tau, int k) { return k < nrt_here && tau >= rows.first[k] && tau < rows.first[k] + rows.count[k]; };
  auto reader = [&](int step, int k) __attribute__((always_inline)) {       // step: of the row tile's own steps
    return make_reader(((step & 1) ? d.ring1 : d.ring0) + (long)rows.tile[k] * nkc * 64, nkc, (n + 3) / 4, wave, lane,
                       ll_fwd_tag((unsigned)step) << 14, err, a.spin_limit, 0);
  };
  // (a loop for slabs of two row tiles and one for a single one: where they met, the compiler would copy loads in flight, behind a wait of its own)
  auto all_steps = [&](auto two) __attribute__((always_inline)) {
  constexpr bool kTwo = decltype(two)::value, kZxAhead = !kTwo && NCH <= 8;
  u32x4 x[NCH];
  auto issue_loads = [&](int tau, int k) __attribute__((always_inline)) {
    const RingReader rn = reader(tau - rows.first[k], k);
#pragma unroll
    for (int it = 0; it < NCH; ++it) x[it] = rn.load_it(it);
  };
  // (a row tile takes part in no step before the longer one of its slab, and in none after it)
  if (kTwo && rows.count[0] > 0) issue_loads(rows.first[0], 0);

  // A single row tile's x W_x + b is fetched a step ahead, behind its ring loads (loads come back in the order of issue: in front of the poll they would hold it
  // up), into LDS, where a wavefront reads back what it asked for: 16 rows of n = 512 2.70 -> 2.50 us a step, of 256 1.99 -> 1.81; wider layers, whose
  // products hide it, lose by it (n = 1024 4.47 -> 4.64).  (Assembly: the compiler makes every later LDS read wait for loads of this kind.)
  auto fetch_zx = [&](int tau) __attribute__((always_inline)) {
    const int t = d.rev ? T - 1 - tau : tau;
    const bool ok = tau < T && active[0] && t < L[0];
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void*)(d.gates + (tau < T ? t : 0) * fg), 0, 0x7ff00000, kBufFlags);
    const unsigned off = ok ? (unsigned)(rows.row[0] * 4 * n + j) * 4u : kParked;
    const unsigned to = zxs_wave + (unsigned)((tau & 1) * sizeof(zxs[0])), gate = (unsigned)n * 4u;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen nt lds" ::"s"(to + (unsigned)(q * sizeof(zxs[0][0][0]))), "v"(off), "s"(rg), "s"(q * gate) : "memory");
  };
  if constexpr (kZxAhead) fetch_zx(0);
  for (int tau = 0; tau < T; ++tau) {
    const int t = d.rev ? T - 1 - tau : tau;
#pragma unroll
    for (int k = 0; k < (kTwo ? 2 : 1); ++k) {             // the slab's row tiles, half a step apart
      PROF_MARK(4)
      const int b = rows.row[k], step = tau - rows.first[k];
      if (!in_loop(tau, k)) {                              // every row of the tile is padding here
        if (kZxAhead && in_loop(tau + 1, 0)) {
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          fetch_zx(tau + 1);
        }
        if (active[k]) {
          ((float*)d.y)[t * fy + (long)b * d.ldy + j] = 0.f;
          if (d.cs) d.cs[t * fs + (long)b * n + j] = c[k];
          if (d.hprev) ((float*)d.hprev)[(t * (long)B + b) * d.ldh + j] = h[k];
        }
        continue;
      }
      const unsigned tagw = ll_fwd_tag((unsigned)step) << 30;
      const bool valid = active[k] && t < L[k];
      // this frame's x W_x + b: in flight while the products run.  In a slab of two row tiles it is asked for when the ring's loads have arrived: their wait is
      // for everything that is in flight (64 rows of n = 1024 8.8 -> 8.2 us a step, 100 of n = 512 5.75 -> 4.85).
      float zx[4];
      const __amdgpu_buffer_rsrc_t zx_rs = __builtin_amdgcn_make_buffer_rsrc((void*)(d.gates + t * fg), 0, 0x7ff00000, kBufFlags);
      const unsigned zx_off = valid ? (unsigned)(b * 4 * n + j) * 4u : kParked;
      auto load_zx = [&]() __attribute__((always_inline)) {
        if constexpr (!kZxAhead) {
#pragma unroll
          for (int q = 0; q < 4; ++q) zx[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zx_rs, zx_off, (unsigned)(q * n) * 4u, 0));      // (marked non-temporal: 4.22 -> 4.91 us a step for 32 rows of n = 1024)
        }
      };
      const RingReader rd = reader(step, k);
      auto next_loads = [&]() __attribute__((always_inline)) {
        if constexpr (kTwo) {
          if (k == 0 && in_loop(tau, 1)) issue_loads(tau, 1);
          else if (in_loop(tau + 1, 0)) issue_loads(tau + 1, 0);
        }
        PROF_MARK(0)
      };
      // accumulator rows 4 * (lane / 16) + v of the row tile, column lane % 16 of the column tile
      auto to_sum = [&](auto&& value) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int v = 0; v < 4; ++v) red[wave][4 * (lane >> 4) + v][ct * 16 + (lane & 15)] = value(ct, v);
      };
      if (__builtin_expect(plain, 0)) {
        f32x4 acc[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
        operands_settle(acc[0], acc[1], acc[2], acc[3]);   // (assembly text: the compiler's own would take accumulation registers from W_h)
#pragma unroll 1
        for (int it = 0; it < NCH; ++it) {
          u32x4 v = rd.load_it(it);
          for (unsigned poll = 0; !dead && __builtin_amdgcn_ballot_w64(rd.tag_diff(v, it, tagw) != 0u) != 0ull; ++poll) {
            if (poll >= a.spin_limit || ((poll & 63u) == 63u && ld_relaxed(err) != 0u)) {
              st_relaxed(err, 1u);
              dead = true;
            }
            v = rd.load_it(it);
          }
          v[1] &= ~kLLFwdTagBit; v[3] &= ~kLLFwdTagBit;
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            const u32x4 wv = w_at(it, ct);
            u32x4 av = v, bv = wv;
            operands_settle(av, bv);
#pragma unroll
            for (int e = 0; e < 4; ++e) mfma4_b_vgpr(acc[ct], __uint_as_float(av[e]), __uint_as_float(bv[e]));
          }
        }
        load_zx();
        next_loads();
        if constexpr (kZxAhead) fetch_zx(tau + 1);
        mfma_settle(acc[0], acc[1], acc[2], acc[3]);
        to_sum([&](int ct, int v) { return acc[ct][v]; });
      } else {
        // Every tag is looked at in front of the products (no branch may come between them: where two paths meet the compiler moves accumulators,
        // and it does not know what is still being written); loads with a stale one are repeated (bounded).  In a slab of two row
        // tiles they went out half a step ago and that is rare; a slab of one waits here for what the half step before published, with two loads, and the others go out then.
        auto fetch = [&](auto from, auto to) __attribute__((always_inline)) {
#pragma unroll
          for (int it = decltype(from)::value; it < decltype(to)::value; ++it) x[it] = rd.load_it(it);
        };
        auto await = [&](auto from, auto to) __attribute__((always_inline)) {
          auto stale = [&]() __attribute__((always_inline)) {
            unsigned bits = 0u;
#pragma unroll
            for (int it = decltype(from)::value; it < decltype(to)::value; ++it) bits |= rd.tag_diff(x[it], it, tagw);
            return __builtin_amdgcn_ballot_w64(bits != 0u) != 0ull;
          };
          if (__builtin_expect(stale() && !dead, 0)) rd.poll_again(dead, [&]() __attribute__((always_inline)) { fetch(from, to); }, stale);
        };
        constexpr std::integral_constant<int, 0> first;
        constexpr std::integral_constant<int, 2> rest;
        constexpr std::integral_constant<int, NCH> all;
        if constexpr (kTwo) {
#pragma unroll
          for (int it = 0; it < NCH; ++it) wait_loads_but(NCH - 1 - it, x[it]);       // (before the stores of the last half step)
          await(first, all);
          load_zx();
        } else {
          if constexpr (!kZxAhead) load_zx();              // (32 rows of n = 1024: 4.27 us a step, 4.70 with these behind the poll)
          fetch(first, rest);
          await(first, rest);
          fetch(rest, all);
          await(rest, all);
          if constexpr (kZxAhead) fetch_zx(tau + 1);
        }
        f32x4 acc[4], low[4];                              // the sum of the largest parts' products, and of the others'
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] = low[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
        operands_settle(acc[0], acc[1], acc[2], acc[3]);   // (the MFMAs are assembly text: wait states by hand)
        operands_settle(low[0], low[1], low[2], low[3]);
        Splitter s[2];
        auto unpack = [&](Splitter& to, int p) __attribute__((always_inline)) {
#pragma unroll
          for (int e = 0; e < 8; ++e) to.v[e] = __uint_as_float(x[2 * p + (e >> 2)][e & 3] & ((e & 1) ? ~kLLFwdTagBit : ~0u));
        };
        unpack(s[0], 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[0].step(e);
        static_for<NP>([&](auto pc) __attribute__((always_inline)) {
          constexpr int p = decltype(pc)::value;
          Splitter &now = s[p & 1], &then = s[(p + 1) & 1];
          __builtin_amdgcn_sched_barrier(0);
          u32x4 wl[4];
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) wl[ct] = w_low[wave][p][ct][lane];
          operands_settle(now.part[0]);
          __builtin_amdgcn_sched_barrier(0);
          // 24 products, and between them the operand's other parts and the next pair's first
#pragma unroll
          for (int o = 0; o < 6; ++o)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) {
              if (o == 0) mfma_b_agpr(acc[ct], now.part[0], wh[p][ct]);
              else if (o == 1) mfma_b_agpr(low[ct], now.part[0], wm[p][ct]);
              else if (o == 2) mfma_b_agpr(low[ct], now.part[1], wh[p][ct]);
              else if (o == 3) mfma_b_agpr(low[ct], now.part[1], wm[p][ct]);
              else if (o == 4) mfma_b_vgpr(low[ct], now.part[0], wl[ct]);
              else mfma_b_agpr(low[ct], now.part[2], wh[p][ct]);
              __builtin_amdgcn_sched_barrier(0);
              const int m = 4 * o + ct;
              if (m < 4) now.step(4 + m);                  // second part, in front of the ninth product
              else if (m >= 8 && m < 12) now.step(m);      // third part, in front of the twenty-first
              if constexpr (p + 1 < NP) {
                if (m == 15) unpack(then, p + 1);
                if (m >= 16 && m < 20) then.step(m - 16);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
        });
        mfma_settle(acc[0], acc[1], acc[2], acc[3]);
        mfma_settle(low[0], low[1], low[2], low[3]);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] += low[ct];
        next_loads();
        to_sum([&](int ct, int v) { return acc[ct][v] * (1.f / kWScale); });
      }
      PROF_MARK(1)
      __syncthreads();
      const float hprev = h[k];
      CellOut o = {};
      if constexpr (kZxAhead) {
#pragma unroll
        for (int q = 0; q < 4; ++q) zx[q] = zxs[tau & 1][wave][q][lane];
      }
      if (valid) {
        float zh[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = col0 + q * 8;
          zh[q] = red[0][r16][col] + red[1][r16][col] + red[2][r16][col] + red[3][r16][col];
        }
        o = lstm_cell(zh, zx, c[k]);
        c[k] = o.c; h[k] = o.h;
      }
      started[k] = started[k] || valid;
      __syncthreads();                // (the accumulators of the other row tile may be written)
      PROF_MARK(2)
      {                               // the recurrence's critical store goes out first (16: agent scope, written through)
        const unsigned h_pub = started[k] ? __float_as_uint(h[k]) : 0u;
        const unsigned h_odd = (unsigned)__builtin_amdgcn_mov_dpp((int)h_pub, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]: the neighbour's h
        // h is below 1 in magnitude, or NaN: a NaN in the tagged half makes its neighbour of the same row NaN instead, as every product with the row is
        const unsigned nan = (unsigned)((int)(h_odd << 1) >> 31);      // bit 30
        const u32x2 unit = {h_pub | nan, (h_odd & ~kLLFwdTagBit) | (ll_fwd_tag((unsigned)step + 1u) << 30)};
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)((step & 1) ? d.ring0 : d.ring1), 0, ring_bytes, kBufFlags);
        const unsigned off = publishes ? (unsigned)rows.tile[k] * (unsigned)nkc * 1024u + pub_in_tile : kParked;
        if (local) __builtin_amdgcn_raw_buffer_store_b64(unit, ro, off, 0, 1);
        else __builtin_amdgcn_raw_buffer_store_b64(unit, ro, off, 0, 16);
      }
      if (active[k]) {                // layer outputs and what the backward pass needs
        ((float*)d.y)[t * fy + (long)b * d.ldy + j] = valid ? h[k] : 0.f;
        if (d.cs) d.cs[t * fs + (long)b * n + j] = c[k];
        if (d.hprev) ((float*)d.hprev)[(t * (long)B + b) * d.ldh + j] = hprev;
        if (valid && a.write_gates) {
          float* gp = d.gates + t * fg + (long)b * 4 * n + j;
          gp[0] = o.gi; gp[n] = o.gf; gp[2 * n] = o.gg; gp[3 * n] = o.go;
        }
      }
      PROF_MARK(3)
    }
  }
  };
  if (nrt_here == 2) all_steps(std::true_type{});
  else all_steps(std::false_type{});
  PROF_DUMP("fwdf32", T)
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (active[k]) {
      const int b = rows.row[k];
      if (d.cT) d.cT[(long)b * n + j] = c[k];
      if (d.hT) d.hT[(long)b * n + j] = h[k];
    }
}

// ------------------------------------------------------------------------------------------------
// backward, float storage: partial sums of Dh, as in the bfloat16 kernels, in the decomposition of the float forward
// kernel (16 units x a slab of 32 rows per work-group, the slab's two row tiles half a step apart).  A work-group
// multiplies ITS dz (16 rows x 64 gate columns, through LDS, never leaving the compute unit) by the matching 64 rows of W_h^T
// for ALL n outputs - 256 registers per lane hold two parts of that slice, LDS the third - and publishes,
// per destination tile of 16 units, the accumulator tile as it stands: a lane's four floats (rows 4g .. 4g+3 of one output)
// are two 8-byte units, the tag bit 30 of each unit's second float.  (Products of three-part sums as forward: 16 k-steps of a column tile are two
// halves of 32 of K.  What the next step's gate gradients need is fetched into LDS a step ahead: loads come back in the order of issue, and from
// memory they would hold up the ring's; n = 512, 32 rows 3.8 -> 3.55 us a step.)  Partial sums are not bounded by 1, so they travel scaled
// by 2^-32 (the consumer multiplies its sum by 2^32): bit 30 is then 0 for every partial
// sum below 2^32 in magnitude, and no other bit of a value above 2^-94 changes.  Larger ones, infinities and NaN travel folded
// (exchange_dev.h): a half step whose largest dz and W_h could make one looks at each sum, the others at none (config 2's loop 525 -> 534 us, a slab of one row
// tile of 1000 units 6.95 -> 7.13 us a step; with a look at every sum 548, with a second copy of the products for such half steps 550, with the
// operands looked at behind the first tiles' MFMAs instead of in front of them 546 and 7.38).  To a consumer a folded value looks like a stale
// tag, and the pass that fetches such loads again unfolds it.  A consumer adds the blocks of its tile from
// all producers (1 KiB each, one 16-byte load per lane: the producer's accumulator layout), wavefront w taking producers
// w, w + 4, ..., and the four sums meet in LDS.
// Ring per direction and slot: [row tile][destination tile][producer tile] x 1 KiB.  K axis of the product: gate column
// kappa = 16 kg + s of the work-group's 64 (gate kappa / 16, unit kappa % 16) is k-step s of lane group kg, so that a lane
// reads its sixteen A values from sixteen consecutive floats of a dz row in LDS.
template <int NCT>                                         // column tiles per wavefront at most: n <= 64 * NCT
__global__ __launch_bounds__(256) void persist_bwd_f32_kernel(PBwdArgs a) {
  __shared__ float red[4][16][17];                         // [wavefront][row][output]
  __shared__ __attribute__((aligned(16))) float zb[16][68];// dz of the row tile in hand: [row][gate column kappa]
  __shared__ u32x4 w_low[4][NCT][2][64];                   // [wavefront][column tile][half of K][lane]
  __shared__ float in_f[2][4][7][64];                      // [row tile][wavefront][gates, cells, dy][lane]: what the next step's gate gradients need
  const WgCoord wg = wg_coord(a.map, a.ndir);
  if (!wg.live) return;
  publish_xcd(a.xcc, wg.base, wg.tile);
  const int J = wg.tile;                                   // tile of 16 units
  const PBwdDir d = a.d[wg.dir];       // a copy: fields read through a reference are fetched again in every time step
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = a.n, B = a.B, T = a.T;
  const int ntile = (n + 15) / 16;
  unsigned* err = a.sync;
  bool dead = false;

  // W_h^T slice: column tile wave + 4 ci of the outputs, k-step s (pack_wh_bwd_f32p_body)
  // In three bfloat16 parts, as forward: two fill the 256 accumulation registers of every lane, the smallest lies in LDS.
  u32x4 wh[NCT][2], wm[NCT][2];
  float w_bound = 0.f;                                     // 64 times the slice's largest weight, over all lanes: a sum of products, scaled by 2^-32, is no larger
  unsigned w_most = 0u;                                    // than this times the largest dz
  auto w_at = [&](int ci, int s4) __attribute__((always_inline)) { return *((const u32x4*)d.Wb + ((((long)J * 4 + wave) * NCT + ci) * 4 + s4) * 64 + lane); };
#pragma unroll
  for (int c2 = 0; c2 < NCT; c2 += 2) {
    u32x4 v[2][4];
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) v[s4 >> 2][s4 & 3] = w_at(c2 + (s4 >> 2), s4 & 3);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int ci = c2 + (g >> 1), c = g & 1;
      Splitter s;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float w = __uint_as_float(v[g >> 1][2 * c + (e >> 2)][e & 3]);
        w_bound = max_magnitude(w_bound, w, 0.f);
        s.v[e] = w * kBwdScale;
        w_most = max(w_most, __float_as_uint(s.v[e]) & 0x7fffffffu);
      }
#pragma unroll
      for (int e = 0; e < 12; ++e) s.step(e);
      wh[ci][c] = s.part[0];
      wm[ci][c] = s.part[1];
      w_low[wave][ci][c][lane] = s.part[2];
      asm volatile("" : "+a"(wh[ci][c]), "+a"(wm[ci][c]));
    }
  }
  const bool plain = __builtin_amdgcn_ballot_w64(w_most >= kWMost) != 0ull;      // (as forward)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) w_bound = max_magnitude(w_bound, __shfl_xor(w_bound, o), 0.f);
  w_bound *= 64.f * kPartScale;
  const int local = NCT <= 8 ? group_is_xcd_local(a.xcc, wg.base, a.map.ntile, a.spin_limit) : 0;      // (more than 32 members never are)

  // pointwise: row r16 of each row tile, unit u of the tile's 16
  const int r16 = tid >> 4, u = tid & 15;
  const int j = J * 16 + u;
  const F32Rows rows = f32_rows(a.lens, B, T, d.rev, a.slab0 + wg.rt, a.slab_tiles, r16);
  const int nrt_here = rows.count_tiles;
  float Dh[2] = {0.f, 0.f}, Dc[2] = {0.f, 0.f};
  float dbsum[4] = {0.f, 0.f, 0.f, 0.f};                    // bias gradient of this thread's unit over its two rows and all frames
  int L[2] = {0, 0};
  bool active[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = rows.row[k];
    active[k] = b >= 0 && j < n;
    if (active[k]) {
      if (d.dhT) Dh[k] = d.dhT[(long)b * n + j];
      if (d.dcT) Dc[k] = d.dcT[(long)b * n + j];
      L[k] = clamp_len(a.lens, b, T);
    }
  }
  const long fg = (long)B * 4 * n, fy = (long)B * d.lddy, fs = (long)B * n;    // elements per frame
  const unsigned ring_bytes = (unsigned)((B + 15) / 16) * (unsigned)ntile * (unsigned)ntile * 1024u;
  PROF_DECL
  // The reader of the partial sums that step sigma consumes for row tile k.  In a slab of two row tiles they are collected
  // DURING the products of the half step before (the other row tile's): what they fetch was published half a step
  // earlier, the loads run kWin ahead of the additions, one load and one addition behind each column tile's MFMAs, and
  // the matrix cores do not wait for the exchange.  `ps_c` / `redo_c` carry the sums (or, if a tag was stale, the order to fetch
  // everything again) into the next half step.
  constexpr int kWin = NCT < 6 ? NCT : 6;
  static_assert(kWin >= 1 && kWin <= 16 && kWin <= NCT, "wait_loads_but covers up to 15 younger loads");
  u32x4 x[NCT < 16 ? 16 : NCT];                            // (an array of up to 128 bytes becomes one register tuple, moved as a whole)
  float ps_c[4] = {0.f, 0.f, 0.f, 0.f};
  unsigned long long redo_c = 0ull;
  bool have_c = false;
  // A row tile's own steps: step s of `count` works on position first + count - 1 - s in processing order; step `count` only
  // collects the Dh that leaves the tile's first frame.  In a shorter tile they begin later (reversed: end earlier).
  auto step_of = [&](int sigma, int k) { return sigma - (T - rows.first[k] - rows.count[k]); };
  auto in_loop = [&](int sigma, int k) { const int st = step_of(sigma, k); return k < nrt_here && st >= 0 && st <= rows.count[k] && rows.count[k] > 0; };
  auto reader = [&](int st, int k) __attribute__((always_inline)) {
    RingReader rd;
    const long tile_base = (((long)rows.tile[k] * ntile + J) * ntile) * 64;                    // uint4 index of [row tile][J][0]
    rd.rs = __builtin_amdgcn_make_buffer_rsrc((void*)((((st - 1) & 1) ? d.ring1 : d.ring0) + tile_base), 0, ntile * 1024, kBufFlags);
    rd.voff = (unsigned)(wave * 1024 + lane * 16);       // load `it` of this wavefront covers producer wave + 4 it
    rd.it_bytes = 4096u;
    rd.lim = ntile - wave; rd.lim_step = 4;
    rd.tag = part_tag(st) << 14; rd.err = err; rd.limit = a.spin_limit;
    rd.nitv = (ntile + 3) / 4; rd.rot = 0;
    return rd;
  };
  auto add_to = [](float (&ps)[4], const u32x4& v) __attribute__((always_inline)) {
    ps[0] += __uint_as_float(v[0]); ps[1] += __uint_as_float(v[1] & ~kLLFwdTagBit);
    ps[2] += __uint_as_float(v[2]); ps[3] += __uint_as_float(v[3] & ~kLLFwdTagBit);
  };

  // Step sigma's inputs of row tile k, fetched a step ahead into LDS, where a wavefront reads back what it asked for.  (Assembly: the compiler makes every
  // later LDS read wait for loads of this kind.)
  const unsigned in_lds = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)&in_f[0][wave][0][0]);
  auto fetch_in = [&](int sigma, int k) __attribute__((always_inline)) {
    constexpr unsigned kParked = 0x7ff00000u;
    const int tau = T - 1 - sigma, t = d.rev ? sigma : tau, tp = d.rev ? t + 1 : t - 1;        // tp: the frame before t in processing order
    const bool frame = tau >= 0, before = tp >= 0 && tp < T;
    const bool on = frame && active[k] && t < L[k];
    const int b = rows.row[k];
    auto from = [&](const void* base, long elements) {
      return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + elements * 4), 0, base ? (int)kParked : 0, kBufFlags);
    };
    const long at = frame ? t : 0;
    const __amdgpu_buffer_rsrc_t rg = from(d.gates, at * fg), rc = from(d.cs, at * fs), rp = from(before ? d.cs : d.c0, before ? tp * fs : 0), ry = from(d.dy, at * fy);
    const unsigned g_off = on ? (unsigned)(b * 4 * n + j) * 4u : kParked, s_off = on ? (unsigned)(b * n + j) * 4u : kParked, y_off = on ? (unsigned)(b * d.lddy + j) * 4u : kParked;
    const unsigned to = in_lds + (unsigned)(k * sizeof(in_f[0])), gate = (unsigned)n * 4u;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // what was there has been read
#pragma unroll
    for (int q = 0; q < 4; ++q)
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen nt lds" ::"s"(to + q * 256u), "v"(g_off), "s"(rg), "s"(q * gate) : "memory");
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(to + 4 * 256u), "v"(s_off), "s"(rc) : "memory");
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(to + 5 * 256u), "v"(s_off), "s"(rp) : "memory");
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen nt lds" ::"s"(to + 6 * 256u), "v"(y_off), "s"(ry) : "memory");
  };
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (in_loop(0, k)) fetch_in(0, k);

  // Steps sigma = 0 .. T-1 work on frames (the last frame in processing order first); step T only collects the Dh that
  // leaves the layer.
  for (int sigma = 0; sigma <= T; ++sigma) {
    const int tau = T - 1 - sigma;                         // position in processing order; -1 in the collecting step
    const int t = d.rev ? T - 1 - tau : tau;               // this step's frame (outside [0, T) in the collecting step)
    const int t_next = d.rev ? t - 1 : t + 1;              // the frame of the step before: where the partial sums come from
#pragma unroll
    for (int k = 0; k < 2; ++k) {                          // the slab's two row tiles, half a step apart
      if (k >= nrt_here) break;                            // (the same in every work-group of the exchange group)
      PROF_MARK(4)
      const int b = rows.row[k], st = step_of(sigma, k);
      if (!in_loop(sigma, k) || (st == rows.count[k] && tau >= 0)) {
        // every row of the tile is padding here; the tile's collecting step falls on such a frame if the tile is reversed and shorter
        if (!in_loop(sigma, k) && in_loop(sigma + 1, k)) fetch_in(sigma + 1, k);
        if (active[k] && tau >= 0) {
          float* zp = (float*)d.DZ + t * fg + (long)b * 4 * n + j;
          zp[0] = 0.f; zp[n] = 0.f; zp[2 * n] = 0.f; zp[3 * n] = 0.f;
        }
        if (!in_loop(sigma, k)) continue;
      }
      const bool pointwise = st < rows.count[k];
      const bool valid = pointwise && active[k] && t < L[k];
      if (st > 0) {                                        // the partial sums of Dh that the step before published
        const RingReader rd = reader(st, k);
        const unsigned tagw = rd.tag << 16;
        const float one = __uint_as_float(kOneBits | tagw);      // (what a magnitude of 1 reads as with the tag in it)
        float ps[4] = {ps_c[0], ps_c[1], ps_c[2], ps_c[3]};
        unsigned long long redo = redo_c;
        if (!have_c) {
          // nothing was collected ahead: a slab of one row tile has no other half step to hide behind (what it consumes
          // is published by the half step before it), and the collecting step follows no products
#pragma unroll
          for (int v = 0; v < 4; ++v) ps[v] = 0.f;
          redo = 0ull;
#pragma unroll
          for (int it = 0; it < NCT; ++it) x[it] = rd.load_it(it);
          float largest = 0.f;
#pragma unroll
          for (int it = 0; it < NCT; ++it) {
            if (__builtin_amdgcn_ballot_w64(rd.tag_diff(x[it], it, tagw) != 0u) == 0ull) {
              add_to(ps, x[it]);
              largest = max_magnitude(largest, __uint_as_float(x[it][1]), __uint_as_float(x[it][3]));
            } else { redo |= 1ull << it; PROF_REDO(1) }
          }
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(largest < one)) != 0ull, 0)) {      // something folded among them: all again
#pragma unroll
            for (int v = 0; v < 4; ++v) ps[v] = 0.f;
            redo = (1ull << NCT) - 1ull;
          }
        }
        if (redo)
          rd.template fix_up_batch<NCT>(redo, dead, [&](int, const u32x4& v) {
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(max_magnitude(0.f, __uint_as_float(v[1]), __uint_as_float(v[3])) < one)) == 0ull, 1)) return add_to(ps, v);
            ps[0] += __uint_as_float(v[0]); ps[1] += __uint_as_float(unfold_wide(v[1] & ~kLLFwdTagBit));
            ps[2] += __uint_as_float(v[2]); ps[3] += __uint_as_float(unfold_wide(v[3] & ~kLLFwdTagBit));
          });
        // a lane's sums: rows 4 (lane / 16) + v of output lane % 16
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][4 * (lane >> 4) + v][lane & 15] = ps[v];
      }
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (elsewhere the ring loads, younger and waited for, say that the inputs are there)
      PROF_MARK(0)
      __syncthreads();
      float in[7];
#pragma unroll
      for (int e = 0; e < 7; ++e) in[e] = in_f[k][wave][e][lane];
      if (st > 0 && active[k] && t_next >= 0 && t_next < L[k])
        Dh[k] = (red[0][r16][u] + red[1][r16][u] + red[2][r16][u] + red[3][r16][u]) * (1.f / kPartScale);
      float dz[4] = {0.f, 0.f, 0.f, 0.f};
      if (valid) lstm_cell_grad(in[0], in[1], in[2], in[3], in[4], in[5], in[6] + Dh[k], Dc[k], dz);
      if (pointwise) {
#pragma unroll
        for (int q = 0; q < 4; ++q) dbsum[q] += dz[q];       // (zero where the frame is padding)
#pragma unroll
        for (int q = 0; q < 4; ++q) zb[r16][q * 16 + u] = dz[q];
        if (active[k]) {
          float* zp = (float*)d.DZ + t * fg + (long)b * 4 * n + j;
          zp[0] = dz[0]; zp[n] = dz[1]; zp[2 * n] = dz[2]; zp[3 * n] = dz[3];
        }
      }
      PROF_MARK(2)
      __syncthreads();
      have_c = false;
      if (pointwise) {
        if (nrt_here == 1) fetch_in(sigma + 1, k);         // (in a slab of two behind the products, whose loads from the ring it would hold up)
        // what the next half step consumes (the other row tile's partial sums, published half a step ago) is collected here
        const int k_n = k ^ 1, sigma_n = k == 0 ? sigma : sigma + 1, st_n = step_of(sigma_n, k_n);
        // (the next half step must be the other tile's, and not its first, which consumes nothing)
        bool collect = in_loop(sigma_n, k_n) && st_n >= 1;
        const RingReader rn = reader(st_n, k_n);
        const unsigned tagw_n = rn.tag << 16;
        float psn[4] = {0.f, 0.f, 0.f, 0.f};
        unsigned stale_n = 0u;
        float largest_n = 0.f;
        if (collect) {
#pragma unroll
          for (int it = 0; it < kWin; ++it) x[it] = rn.load_it(it);
        }
        // A operand: row lane % 16, gate columns 16 (lane / 16) .. + 15
        float av[16];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const float4 v = *(const float4*)&zb[lane & 15][(lane >> 4) * 16 + 4 * s4];
          av[4 * s4] = v.x; av[4 * s4 + 1] = v.y; av[4 * s4 + 2] = v.z; av[4 * s4 + 3] = v.w;
        }
        const unsigned tag_hi = part_tag(st + 1) << 30;
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)((st & 1) ? d.ring1 : d.ring0), 0, ring_bytes, kBufFlags);
        // destination tile wave + 4 ci (one past the last: parked), this producer's block
        const unsigned pub0 = (unsigned)(((rows.tile[k] * ntile + wave) * ntile + J) * 1024 + lane * 16);
        // The accumulator of column tile ci is published behind the MFMAs of column tile ci + 1: by then its last MFMA has long
        // finished (the compiler does not see the MFMAs in the assembly text and inserts no wait states for their results).
        // Could a sum of 64 products not be below 1?  Asked of the operands, once per half step.  Then the same code leaves the sums as they
        // are in this work-group's part of d.wide, and they are folded on their way from there.
        float largest = 0.f;
#pragma unroll
        for (int s = 0; s < 16; s += 2) largest = max_magnitude(largest, av[s], av[s + 1]);
        // (scalar arithmetic by hand: a choice between two descriptors is applied lane by lane)
        const unsigned long long which = 0ull - (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(__builtin_amdgcn_ballot_w64(is_wide(largest * w_bound)) != 0ull);
        const bool wide = which != 0ull;
        const unsigned long long ring = (unsigned long long)((st & 1) ? d.ring1 : d.ring0);
        const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc((void*)(ring ^ ((ring ^ (unsigned long long)d.wide) & which)), 0, ring_bytes, kBufFlags);
        const unsigned mark = tag_hi & ~(unsigned)which;
        auto publish = [&](int ci, const f32x4& acc) __attribute__((always_inline)) {
          const u32x4 unit = {__float_as_uint(acc[0]), __float_as_uint(acc[1]) | mark, __float_as_uint(acc[2]), __float_as_uint(acc[3]) | mark};
          const unsigned off = wave + 4 * ci < ntile ? pub0 + (unsigned)(4 * ci) * (unsigned)ntile * 1024u : 0x7ff00000u;
          if (local) __builtin_amdgcn_raw_buffer_store_b128(unit, to, off, 0, 1);
          else __builtin_amdgcn_raw_buffer_store_b128(unit, to, off, 0, 16);    // 16: agent scope, written through
        };
        // What the parts or, scaled by 2^48, their sums cannot hold: float MFMAs, W_h from memory, and the next half step fetches for itself.
        const float bound = largest * w_bound;
        if (__builtin_expect(plain || __builtin_amdgcn_ballot_w64(!(largest < 0x1p100f && bound < 0x1p44f)) != 0ull, 0)) {
          collect = false;
#pragma unroll 1
          for (int ci = 0; ci < NCT; ++ci) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, o1 = acc, o2 = acc, o3 = acc;
            operands_settle(acc, o1, o2, o3);
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
              u32x4 wv = w_at(ci, s4), none = wv;
#pragma unroll
              for (int e = 0; e < 4; ++e) wv[e] = __float_as_uint(__uint_as_float(wv[e]) * kPartScale);
              operands_settle(wv, none);
#pragma unroll
              for (int e = 0; e < 4; ++e) mfma4_b_vgpr(acc, av[4 * s4 + e], __uint_as_float(wv[e]));
            }
            mfma_settle(acc);
            publish(ci, acc);
          }
        } else {
          Splitter s[2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s[c].v[e] = av[8 * c + e] * kBwdScale;
#pragma unroll
            for (int e = 0; e < 12; ++e) s[c].step(e);
          }
          u32x4 wl[2][2];
#pragma unroll
          for (int c = 0; c < 2; ++c) wl[0][c] = w_low[wave][0][c][lane];
          operands_settle(s[0].part[0], s[0].part[1], s[0].part[2], s[1].part[0]);
          operands_settle(s[1].part[1], s[1].part[2]);
          f32x4 acc2[2], low2[2];                          // (low: the products of all but the largest parts)
#pragma unroll
          for (int ci = 0; ci < NCT; ++ci) {
            f32x4 &acc = acc2[ci & 1], &low = low2[ci & 1];
            __builtin_amdgcn_sched_barrier(0);
            if (ci + 1 < NCT) {
#pragma unroll
              for (int c = 0; c < 2; ++c) wl[(ci + 1) & 1][c] = w_low[wave][ci + 1][c][lane];
            }
            __builtin_amdgcn_sched_barrier(0);
            mfma_b_agpr_first(acc, s[0].part[0], wh[ci][0]);
            mfma_b_agpr_first(low, s[0].part[0], wm[ci][0]);
            mfma_b_agpr(acc, s[1].part[0], wh[ci][1]);
            mfma_b_agpr(low, s[1].part[0], wm[ci][1]);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              mfma_b_agpr(low, s[c].part[1], wh[ci][c]);
              mfma_b_agpr(low, s[c].part[1], wm[ci][c]);
              mfma_b_agpr(low, s[c].part[2], wh[ci][c]);
              mfma_b_vgpr(low, s[c].part[0], wl[ci & 1][c]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ci > 0) publish(ci - 1, (acc2[(ci - 1) & 1] + low2[(ci - 1) & 1]) * kSumScale);
            if (collect) {                                 // (behind the MFMAs just issued: they run while this does)
              wait_loads_but((NCT - 1 - ci) < (kWin - 1) ? (NCT - 1 - ci) : (kWin - 1), x[ci % kWin]);     // the younger loads: the window's others
              stale_n |= rn.tag_diff(x[ci % kWin], ci, tagw_n);      // looked at once, behind the last load
              largest_n = max_magnitude(largest_n, __uint_as_float(x[ci % kWin][1]), __uint_as_float(x[ci % kWin][3]));
              add_to(psn, x[ci % kWin]);
              if (ci + kWin < NCT) x[ci % kWin] = rn.load_it(ci + kWin);
            }
          }
          mfma_settle(acc2[(NCT - 1) & 1]);
          mfma_settle(low2[(NCT - 1) & 1]);
          publish(NCT - 1, (acc2[(NCT - 1) & 1] + low2[(NCT - 1) & 1]) * kSumScale);
        }
        if (__builtin_expect(wide, 0)) {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (a wavefront reads what it stored itself, past its L1)
#pragma unroll 1
          for (int c = wave; c < ntile; c += 4) {
            const unsigned off = pub0 + (unsigned)(c - wave) * (unsigned)ntile * 1024u;
            u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(to, off, 0, kSc1);
            v[1] = fold_wide(v[1]) | tag_hi;
            v[3] = fold_wide(v[3]) | tag_hi;
            if (local) __builtin_amdgcn_raw_buffer_store_b128(v, ro, off, 0, 1);
            else __builtin_amdgcn_raw_buffer_store_b128(v, ro, off, 0, 16);
          }
        }
        if (nrt_here == 2) fetch_in(sigma + 1, k);
        if (collect) {
          // The tags are looked at once, here: a test and a branch per load cost a twentieth of the step.  A stale tag anywhere
          // (a tenth of the half steps): the sums are dropped and the next half step fetches every load again.
          const bool again = __builtin_amdgcn_ballot_w64((stale_n != 0u) | !(largest_n < __uint_as_float(kOneBits | tagw_n))) != 0ull;
          if (again) { PROF_REDO(NCT) }
#pragma unroll
          for (int v = 0; v < 4; ++v) ps_c[v] = again ? 0.f : psn[v];
          redo_c = again ? (1ull << NCT) - 1ull : 0ull;
          have_c = true;
        }
      }
      PROF_MARK(1)
    }
  }
  PROF_DUMP("bwdf32", T)
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (active[k]) {
      const int b = rows.row[k];
      if (d.dh0) d.dh0[(long)b * n + j] = Dh[k];
      if (d.dc0) d.dc0[(long)b * n + j] = Dc[k];
    }
  if (d.dbpart) {                       // bias gradient: this work-group's rows summed into the first slice of its first row tile (the others stay zero)
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) zb[r16][q * 16 + u] = dbsum[q];
    __syncthreads();
    if (tid < 64) {
      const int q = tid >> 4, uu = tid & 15, jj = J * 16 + uu;
      float sum = 0.f;
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) sum += zb[rr][q * 16 + uu];
      if (jj < n) d.dbpart[(long)2 * rows.tile[0] * 4 * n + q * n + jj] = sum;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// packing for the ring layout
// forward weights: chunk index = (((dir*ntile + tile)*4 + q)*nkc + kc)*64 + lane, or (`paired`: the 8-row kernel)
// ((((dir*ntile2 + tile2)*4 + q)*nkc + kc)*2 + set)*64 + lane, two column tiles in one operand (smfmac_b_agpr)
__device__ __forceinline__ void pack_wh_fwd_ll_body(long idx, const bf16_t* W, uint4* out, int n, int nkc, int paired, long total) {
  if (idx >= total) return;
  const int lane = idx & 63, g = lane >> 4;
  long rest = idx >> 6;
  int set = 0;
  if (paired) { set = rest & 1; rest >>= 1; }
  const int kc = rest % nkc; rest /= nkc;
  const int q = rest & 3; rest >>= 2;
  const int ntile = ((n + 31) / 32) << (paired ? 0 : 1);   // (as many bytes either way)
  const int tile = rest % ntile, dir = rest / ntile;
  const bf16_t* Wd = W + (long)dir * n * 4 * n;
  bf16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // forward ring: slot = unit index (kLLSlotsFwd = kLLValsFwd)
    const int k = kc * 32 + (paired ? sparse_k(set, g, e) : g * 8 + e);
    const int j = (paired ? tile * 32 + 16 * sparse_tile(e) : tile * 16) + (lane & 15);
    v[e] = (k < n && j < n) ? Wd[(long)k * 4 * n + q * n + j] : (bf16_t)0.f;
  }
  out[idx] = *(uint4*)v;
}
// partial-sum backward kernels: chunk index = ((((dir*ntile2 + J)*4 + wave)*4 + kc)*nct + c)*64 + lane ; B fragment of
// gate kc, K = the 32 units of tile J, columns = outputs (wave*nct + c)*16 .. +15: eight consecutive units of a row of W_h, or
// (`paired`: the 8-row kernel, c = 2P + set) four consecutive ones of two rows 16 apart, two by two (smfmac_b_agpr).
// (16-byte reads: the set-up of config 3's backward loops, with its fills, 27 -> 17 us.)  Scaled by 2^-32, exactly: the partial sums of Dh leave the MFMAs scaled, which keeps a bit of their bf16 form free.
__device__ __forceinline__ void pack_wh_bwdp_body(long idx, const bf16_t* W, uint4* out, int n, int ntile2, int nct, int paired, long total) {
  if (idx >= total) return;
  const int lane = idx & 63, g = lane & 3, col = lane >> 2;  // (four neighbouring threads read 64 consecutive bytes)
  long rest = idx >> 6;
  const int c = rest % nct; rest /= nct;
  const int kc = rest & 3, wave = (rest >> 2) & 3;
  rest >>= 4;
  const int J = rest % ntile2, dir = rest / ntile2;
  const uint16_t* Wd = (const uint16_t*)W + (long)dir * n * 4 * n + kc * n;
  auto scaled = [](unsigned bits) { return (unsigned)f2bf_bits(bf_bits2f((uint16_t)bits) * kPartScale); };
  unsigned v[8];
  if (paired) {
    const int u0 = J * 32 + sparse_k(c & 1, g, 0);           // elements 0, 1, 4, 5: u0 .. u0 + 3 of the first row; 2, 3, 6, 7: of the second
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int jout = (wave * nct + (c & ~1) + h) * 16 + col;
      const uint16_t* p = Wd + (long)min(jout, n - 1) * 4 * n;
      unsigned x[4];
      if (n % 4 == 0) {
        const uint2 y = *(const uint2*)(p + min(u0, n - 4));
        x[0] = y.x & 0xffffu; x[1] = y.x >> 16; x[2] = y.y & 0xffffu; x[3] = y.y >> 16;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = p[min(u0 + e, n - 1)];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[(e & 1) + 2 * h + 4 * (e >> 1)] = jout < n && u0 + e < n ? scaled(x[e]) : 0u;
    }
  } else {
    const int u0 = J * 32 + g * 8, jout = (wave * nct + c) * 16 + col;
    const uint16_t* p = Wd + (long)min(jout, n - 1) * 4 * n;
    if (n % 8 == 0) {
      const uint4 x = *(const uint4*)(p + min(u0, n - 8));
      v[0] = x.x & 0xffffu; v[1] = x.x >> 16; v[2] = x.y & 0xffffu; v[3] = x.y >> 16; v[4] = x.z & 0xffffu; v[5] = x.z >> 16; v[6] = x.w & 0xffffu; v[7] = x.w >> 16;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p[min(u0 + e, n - 1)];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = jout < n && u0 + e < n ? scaled(v[e]) : 0u;
  }
  out[(idx & ~63l) + g * 16 + col] = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}
// Initial contents of the forward ring, one 8-byte unit per thread: slot 0 = zeros that carry the tag of step 0, slot 1 = zeros.
__device__ __forceinline__ void pack_state_ll_body(long idx, uint4* ring0, uint4* ring1, long total) {
  if (idx >= total) return;
  ((unsigned long long*)ring0)[idx] = (unsigned long long)(ll_fwd_tag(0u) * kLLFwdTagBit) << 32;
  ((unsigned long long*)ring1)[idx] = 0ull;
}
// Everything a bfloat16 single-launch loop needs set up, in ONE launch (three kernels in a row cost three start-ups and run one
// after the other; none of them depends on another): blocks [0, first_pack) clear the regions of `z` (as fill_zero_many_kernel does),
// blocks [first_pack, first_ring) bring W_h into the kernel's order (forward: ring order; backward: the partial-sum kernel's),
// blocks [first_ring, first_map) (forward only) write the initial ring, blocks from first_map on number the real frames
// (frame_map_body) when the products that follow go over real frames only.
// Are rows one behind the other faster?  The same for every wavefront of a launch: about as many steps as the table will have (more than the
// average place or the longest row only where few long rows are left for the end).
__device__ __forceinline__ bool rows_pay(const PackRows& p) {
  int sum = 0, most = 0;
  for (int b = threadIdx.x & 63; b < p.B; b += 64) {
    const int L = clamp_len(p.lens, b, p.T);
    sum += L;
    most = max(most, L);
  }
#pragma unroll
  for (int o = 32; o; o >>= 1) {
    sum += __shfl_xor(sum, o);
    most = max(most, __shfl_xor(most, o));
  }
  return __builtin_amdgcn_readfirstlane(max(most, (sum + p.slots - 1) / p.slots)) <= p.max_steps;
}
// The table of rows one behind the other (see RowTable), by one block: rows by falling length, each to the place with the fewest
// frames so far (the first `slots` rows start a place each).  Two tables, frames ascending and descending in time; B <= 256.
__device__ __forceinline__ void pack_rows_body(const PackRows& p) {
  __shared__ int len[256], order[256], start[256], place[256], total[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (!rows_pay(p)) {
    if (tid == 0) p.steps[0] = -1;
    return;
  }
  if (tid < p.B) len[tid] = clamp_len(p.lens, tid, p.T);
  __syncthreads();
  if (tid < p.B) {
    const int L = len[tid];
    int rank = 0;
    for (int b = 0; b < p.B; ++b) rank += len[b] > L || (len[b] == L && b < tid);
    order[rank] = tid;
  }
  __syncthreads();
  if (wave == 0) {                                         // one wavefront: places (lane + 64 i) and rows (rank lane + 64 i) in registers
    int sum[4], row[4], rlen[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = lane + 64 * i;
      row[i] = k < p.B ? order[k] : 0;
      rlen[i] = k < p.B ? len[row[i]] : 0;
      sum[i] = k < p.slots ? (k < p.B ? rlen[i] : 0) : 0x7fffff;
      if (k < p.slots && k < p.B) { place[row[i]] = k; start[row[i]] = 0; }
    }
    for (int k = p.slots; k < p.B; ++k) {
      const int i = k >> 6;
      const int b = __builtin_amdgcn_readlane(i == 0 ? row[0] : i == 1 ? row[1] : i == 2 ? row[2] : row[3], k & 63);
      const int L = __builtin_amdgcn_readlane(i == 0 ? rlen[0] : i == 1 ? rlen[1] : i == 2 ? rlen[2] : rlen[3], k & 63);
      unsigned best = ~0u;                                 // frames so far (below 2^23) and place
#pragma unroll
      for (int j = 0; j < 4; ++j) best = min(best, ((unsigned)sum[j] << 8) | (unsigned)(lane + 64 * j));
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x111, 0xf, 0xf, false));   // row_shr 1, 2, 4, 8; row_bcast 15, 31
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x112, 0xf, 0xf, false));
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x114, 0xf, 0xf, false));
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x118, 0xf, 0xf, false));
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x142, 0xa, 0xf, false));
      best = min(best, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)best, 0x143, 0xc, 0xf, false));
      const unsigned won = (unsigned)__builtin_amdgcn_readlane((int)best, 63);
      const int q = (int)(won & 255u), before = (int)(won >> 8);
      if (lane == 0) { place[b] = q; start[b] = before; }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (lane + 64 * j == q) sum[j] += L;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (lane + 64 * j < p.slots) total[lane + 64 * j] = sum[j];
  }
  __syncthreads();
  for (int b = wave; b < p.B; b += 4) {
    const int L = len[b], q = place[b];
    const long at = ((long)(q >> 3) * p.tab_steps + start[b]) * 8 + (q & 7);
    for (int i = lane; i < L; i += 64) {
      const unsigned flags = kRowValid | (i == 0 ? kRowFirst : 0u) | (i == L - 1 ? kRowLast : 0u);
      p.up[at + (long)i * 8] = (unsigned)(i * p.B + b) | flags;
      p.down[at + (long)i * 8] = (unsigned)((L - 1 - i) * p.B + b) | flags;
    }
  }
  for (int q = wave; q < p.slots; q += 4) {                // places that are done before their group is
    int most = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) most = max(most, total[(q & ~7) + r]);
    if (lane == 0 && (q & 7) == 0) p.steps[q >> 3] = most;
    for (int i = total[q] + lane; i < most; i += 64) {
      const long at = ((long)(q >> 3) * p.tab_steps + i) * 8 + (q & 7);
      p.up[at] = 0u;
      p.down[at] = 0u;
    }
  }
}
// What the loops leave out where rows run one behind the other: y = 0 and the carried cell state at padded frames.  A wavefront takes
// a frame, 16 bytes a lane where rows allow it.
struct FillArgs { const int* lens; const int* steps; int T, B, n, ndir; uint16_t* y; float* cs[2]; const float* c0[2]; int rev[2]; int vec_y, vec_c; };
__global__ __launch_bounds__(256) void fill_padded_kernel(FillArgs a) {
  const int b = blockIdx.x, t = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int L = clamp_len(a.lens, b, a.T);
  if (t < L || t >= a.T || a.steps[0] < 0) return;
  const long row = (long)t * a.B + b, width = (long)a.ndir * a.n;         // (n is even: whole words)
  const float* src[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
    src[d] = d < a.ndir && a.cs[d] ? !a.rev[d] && L > 0 ? a.cs[d] + ((long)(L - 1) * a.B + b) * a.n : a.c0[d] ? a.c0[d] + (long)b * a.n : nullptr : nullptr;
  // n <= 1024 (persist_pack_slots): four pieces of a lane are a row's, all asked for before anything is stored (one at a time was a chain of up to eight
  // latencies: 64 rows of 20 - 80 frames, n = 1000, both directions 8.7 us, now 7.4)
  float4 v[2][4];
  if (a.vec_c) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[d][k] = src[d] ? ((const float4*)src[d])[min(lane + 64 * k, a.n / 4 - 1)] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (a.vec_y) {
    uint4* y = (uint4*)(a.y + row * width);
    for (int i = lane; i < width / 8; i += 64) y[i] = make_uint4(0, 0, 0, 0);
  } else {
    unsigned* y = (unsigned*)(a.y + row * width);
    for (int i = lane; i < width / 2; i += 64) y[i] = 0u;
  }
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    if (d >= a.ndir || !a.cs[d]) continue;
    float* dst = a.cs[d] + row * a.n;
    if (a.vec_c) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (lane + 64 * k < a.n / 4) ((float4*)dst)[lane + 64 * k] = v[d][k];
    } else {
      for (int i = lane; i < a.n; i += 64) dst[i] = src[d] ? src[d][i] : 0.f;
    }
  }
}
struct PrepArgs {
  ZeroRegions z;
  const bf16_t* W; uint4* Wout; int n, nk, nct; long w_total;   // nk: nkc (forward) / ntile2 (backward)
  uint4* ring0; uint4* ring1; long ring_total;
  const int* lens; int T, B; int* fidx; int* count;     // frame map (fidx == NULL: none)
  PackRows rows;                                          // rows one behind the other: one more block (slots > 0)
  SetUpCopies copies;
  int first_pack, first_ring, first_pad, first_h0, first_map, backward, paired;
};
// Blocks of the copies: [first_pad, first_h0) x, [first_h0, first_map) the initial state.
template <typename TW>
__device__ __forceinline__ void copies_body(const SetUpCopies& c, int block, int pad_blocks, int tid) {
  if (block < pad_blocks) {
    pad_rows_body((long)block * 256 + tid, (const uint16_t*)c.x, (uint4*)c.xpad, c.x_rows, c.x_cols, c.x_ld / 8);
    return;
  }
  const long idx = (long)(block - pad_blocks) * 256 + tid;
  if (idx >= (long)c.ndir * c.B * c.ld) return;
  const long r = idx / c.ld;
  const int k = (int)(idx - r * c.ld), dir = r >= c.B, b = (int)r - dir * c.B;
  if (k == 0) {
    const int L = clamp_len(c.lens, b, c.T);
    c.row[r] = ((dir == 0 ? c.rev0 : c.rev1) && L > 0 ? L - 1 : 0) * c.B + b;
  }
  const float v = k < c.n ? c.h0[r * c.n + k] : 0.f;
  if constexpr (sizeof(TW) == 2) ((uint16_t*)c.out)[idx] = f2bf_bits(v);
  else ((float*)c.out)[idx] = v;
}
constexpr int kTouch = 4;
__device__ __forceinline__ void set_up_body(const PrepArgs& a, int bid, int tid) {       // (256 threads, no frame map)
  if (bid < a.first_pack) {
    fill_zero_body(a.z, bid, tid);
  } else if (bid < a.first_ring) {
    const long idx = (long)(bid - a.first_pack) * 256 + tid;
    if (!a.Wout) {                                         // the loop takes W_h as it is: fetched, for it to be in the last-level cache by then
      const unsigned* W = (const unsigned*)a.W;            // (a word of every 64 bytes; here by the whole device, there by the XCDs of the loop)
      unsigned v[kTouch];
#pragma unroll
      for (int t = 0; t < kTouch; ++t) v[t] = W[min((((long)(bid - a.first_pack) * kTouch + t) * 256 + tid) * 16, a.w_total - 1)];
#pragma unroll
      for (int t = 0; t < kTouch; ++t) asm volatile("" ::"v"(v[t]));
      return;
    }
    const int paired = a.rows.slots > 0 ? rows_pay(a.rows) : a.paired;
    if (a.backward) pack_wh_bwdp_body(idx, a.W, a.Wout, a.n, a.nk, a.nct, paired, a.w_total);
    else pack_wh_fwd_ll_body(idx, a.W, a.Wout, a.n, a.nk, paired, a.w_total);
  } else if (bid < a.first_pad) {
    pack_state_ll_body((long)(bid - a.first_ring) * 256 + tid, a.ring0, a.ring1, a.ring_total);
  } else if (bid < a.first_map) {
    copies_body<bf16_t>(a.copies, bid - a.first_pad, a.first_h0 - a.first_pad, tid);
  }
}
__global__ __launch_bounds__(256) void prep_ll_kernel(PrepArgs a) {
  if (a.rows.slots > 0 && blockIdx.x == 0) {               // (a chain of its own: the longest, so it starts first)
    pack_rows_body(a.rows);
    return;
  }
  const int bid = (int)blockIdx.x - (a.rows.slots > 0 ? 1 : 0);
  if (bid < a.first_map) set_up_body(a, bid, threadIdx.x);
  else frame_map_body(bid - a.first_map, a.lens, a.T, a.B, a.fidx, a.count);
}
// A short batch: the input projection of all frames (few_zx_ok; padded ones too: nobody reads what they get) together with the set-up, which
// it has nothing to do with.  The product is a read of W_x (32 MB at n_in = 2000, n = 1000, two directions).  As it lies in memory W_x has a row's units
// side by side where MFMA wants a unit's k: a lane fetches kFewUnits units of eight rows and turns them in registers, after which
// it holds the operands of that many products, unit kFewUnits i + h of lane i's being column i of product h.  So nothing is staged.
// A work-group owns 32 units, its eight wavefronts share the chunks of 32 k, two chunks in flight each; their sums meet in LDS.
// What bounds it is how much a compute unit has in flight, so it is narrow tiles that count: with 128 units a work-group (63 of them, 16-byte loads)
// the launch took 20.0 us, with 64 16.2, with 32 (250 work-groups, 64 bytes of a row) 15.5; two to four chunks in flight the same, more slower.  Before: set-up
// 11.8 us (most of it packing W_h), the product in K ranges 12.6, their sum 4.8.
struct FewZxArgs { const uint16_t* x; const uint16_t* W; const float* bias; float* C; int M, K, N, tiles, ndir, blocks; long sC; };
constexpr int kFewWaves = 8, kFewUnits = 2, kFewRing = 2;
template <int MT>
__device__ __forceinline__ void few_zx_body(const FewZxArgs& a, int block, f32x4 (&part)[kFewWaves][MT][kFewUnits][64]) {
  constexpr int P = kFewUnits, kCols = 16 * P;             // (a lane's units: one word)
  const int tile = block % a.tiles, dir = block / a.tiles % a.ndir, r0 = block / a.tiles / a.ndir * 16 * MT, tid = threadIdx.x, lane = tid & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), M = a.M, K = a.K, N = a.N;
  constexpr unsigned kParked = 0x7ff00000u;
  const unsigned ldw = 2u * N, col = tile * kCols + i * P;
  const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.W + (long)dir * K * N), 0, (unsigned)K * ldw, kBufFlags);   // (rows past K: outside)
  const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, (unsigned)M * K * 2u, kBufFlags);
  const unsigned w0 = col < (unsigned)N ? g * 8 * ldw + col * 2u : kParked;
  const int chunks = (K + 31) / 32;
  unsigned w[kFewRing][8];
  u32x4 x[kFewRing][MT];
  auto fetch = [&](int c, unsigned (&wv)[8], u32x4 (&xv)[MT]) __attribute__((always_inline)) {
    const unsigned k0 = c * 32 + g * 8;
#pragma unroll
    for (int m = 0; m < MT; ++m)
      xv[m] = __builtin_amdgcn_raw_buffer_load_b128(x_rs, r0 + m * 16 + i < M && k0 < (unsigned)K ? ((r0 + m * 16 + i) * (unsigned)K + k0) * 2u : kParked, 0, 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) wv[e] = __builtin_amdgcn_raw_buffer_load_b32(w_rs, w0 + (c * 32 + e) * ldw, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4 acc[MT][P];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int h = 0; h < P; ++h) acc[m][h] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < kFewRing; ++s) fetch(wave + s * kFewWaves, w[s], x[s]);
  for (int c = wave; c < chunks; c += kFewRing * kFewWaves) {            // (past the last chunk: zeros, which no memory is read for)
#pragma unroll
    for (int s = 0; s < kFewRing; ++s) {
      const int k0 = (c + s * kFewWaves) * 32 + g * 8;
#pragma unroll
      for (int m = 0; m < MT; ++m)                         // (the last piece of a row may reach into the next)
#pragma unroll
        for (int d = 0; d < 4; ++d) x[s][m][d] = k0 + 2 * d < K ? x[s][m][d] : 0u;
#pragma unroll
      for (int h = 0; h < P; ++h) {
        const unsigned sel = h & 1 ? 0x07060302u : 0x05040100u;          // the high, the low halves of two words
        u32x4 b;
#pragma unroll
        for (int d = 0; d < 4; ++d) b[d] = __builtin_amdgcn_perm(w[s][2 * d + 1], w[s][2 * d], sel);
#pragma unroll
        for (int m = 0; m < MT; ++m)
          acc[m][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[s][m]), __builtin_bit_cast(bf16x8, b), acc[m][h], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      fetch(c + (s + kFewRing) * kFewWaves, w[s], x[s]);
    }
  }
  // Sums: a thread takes (row tile, product, lane).
  constexpr int kSums = MT * P * 64;
  static_assert(kSums <= 512, "a sum each");
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int h = 0; h < P; ++h) part[wave][m][h][lane] = acc[m][h];
  __syncthreads();
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  if (tid < kSums) {
#pragma unroll
    for (int v = 0; v < kFewWaves; ++v) sum += (&part[0][0][0][0])[v * kSums + tid];
  }
  __syncthreads();
  float* out = (float*)&part[0][0][0][0];                  // [row][kOut]: turned into rows
  constexpr int kOut = kCols + 4;
  static_assert(MT * 16 * kOut * 4 <= (int)sizeof(part), "the result must fit");
  if (tid < kSums) {
#pragma unroll
    for (int v = 0; v < 4; ++v) out[(tid / (64 * P) * 16 + (lane >> 4) * 4 + v) * kOut + (lane & 15) * P + wave % P] = sum[v];
  }
  __syncthreads();
  for (int at = tid; at < MT * 4 * kCols; at += 512) {
    const int row = at / (kCols / 4), c1 = at % (kCols / 4) * 4, c0 = tile * kCols + c1;
    if (r0 + row >= M || c0 >= N) continue;                     // (N is a multiple of four)
    float4 v = *(const float4*)&out[row * kOut + c1];
    if (a.bias) {
      const float* b = a.bias + (long)dir * N + c0;
      v.x += b[0]; v.y += b[1]; v.z += b[2]; v.w += b[3];
    }
    *(float4*)(a.C + dir * a.sC + (long)(r0 + row) * N + c0) = v;
  }
}
template <int MT>
__global__ __launch_bounds__(512) void prep_zx_kernel(PrepArgs a, FewZxArgs f) {
  __shared__ f32x4 part[kFewWaves][MT][kFewUnits][64];
  if ((int)blockIdx.x < f.blocks) { few_zx_body<MT>(f, blockIdx.x, part); return; }
  const int bid = ((int)blockIdx.x - f.blocks) * 2 + (threadIdx.x >> 8);
  if (bid < a.first_map) set_up_body(a, bid, threadIdx.x & 255);
}
// Everything a float single-launch loop needs set up, in one launch, as prep_ll_kernel does for bfloat16: as kernels of their own (fills, W_h, the rings of either direction, the
// frame map) they took 4 to 5 us each, most of it the gap (five layers of 896 units, 4 rows of 9 frames, training 1049 -> 983 us).
struct PrepF32Args {
  ZeroRegions z;
  const float* W; void* Wout; int n, nk, nct; long w_total;     // nk: nkc (forward) / unit tiles (backward)
  uint4* ring0[2]; uint4* ring1[2]; long ring_total;            // forward: 16-byte units of a direction's ring
  const int* lens; int T, B; int* fidx; int* count;             // frame map (fidx == NULL: none)
  SetUpCopies copies;
  int first_pack, first_ring, first_pad, first_h0, first_map, per_ring, backward;
};
// W_h^T for the float partial-sum backward kernel: float index
// ((((dir*ntile + J)*4 + wave)*NCT + ci)*16 + s)*64 + lane holds W_h[unit (wave + 4 ci)*16 + lane%16][gate column
// (kappa/16)*n + J*16 + kappa%16], kappa = 16 (lane/16) + s; stored so that a lane's k-steps 4 s4 .. 4 s4 + 3 are one float4:
// float4 index ((((dir*ntile + J)*4 + wave)*NCT + ci)*4 + s4)*64 + lane.
// A wavefront packs one (J, wave, ci): four lanes read the 64 consecutive bytes of a row and gate, and store 256 consecutive bytes with
// the lanes of the other rows (one value per thread and 64 rows per load: 32 us for config 2's two directions).
typedef float4 __attribute__((aligned(4))) float4_u;
__device__ __forceinline__ void pack_wh_bwd_f32p_body(long idx, const float* W, float4* out, int n, int ntile, int nct, long total) {
  if (idx >= total) return;
  const int r = (idx & 63) >> 2, s4 = idx & 3;
  long rest = idx >> 6;
  const int ci = rest % nct; rest /= nct;
  const int wave = rest & 3; rest >>= 2;
  const int J = rest % ntile, dir = rest / ntile;
  const int unit_in = (wave + 4 * ci) * 16 + r, unit_out = J * 16 + 4 * s4;    // kappa = 16 q + s: gate q of unit J * 16 + s
  const float* row = W + ((long)dir * n + min(unit_in, n - 1)) * 4 * n;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (unit_in < n && unit_out + 4 <= n) {                     // (at any float)
      const float4 x = *(const float4_u*)(row + q * n + unit_out);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else if (unit_in < n) {
      for (int e = 0; e < 4; ++e)
        if (unit_out + e < n) v[e] = row[q * n + unit_out + e];
    }
    out[((idx >> 6) * 4 + s4) * 64 + q * 16 + r] = make_float4(v[0], v[1], v[2], v[3]);
  }
}
__global__ __launch_bounds__(256) void prep_f32_kernel(PrepF32Args a) {
  const int bid = blockIdx.x, tid = threadIdx.x;
  if (bid < a.first_pack) {
    fill_zero_body(a.z, bid, tid);
  } else if (bid < a.first_ring) {
    const long idx = (long)(bid - a.first_pack) * 256 + tid;
    if (a.backward) pack_wh_bwd_f32p_body(idx, a.W, (float4*)a.Wout, a.n, a.nk, a.nct, a.w_total);
    else pack_wh_fwd_body(idx, a.W, (uint4*)a.Wout, a.n, a.nk, a.w_total);
  } else if (bid < a.first_pad) {                               // before the first step: slot 0 holds zeros that carry the tag of step 0 in every unit, slot 1 is cleared
    const int d = (bid - a.first_ring) / a.per_ring;
    const long idx = (long)(bid - a.first_ring - d * a.per_ring) * 256 + tid;
    if (idx >= a.ring_total) return;
    const unsigned t = ll_fwd_tag(0u) << 30;
    a.ring0[d][idx] = make_uint4(0u, t, 0u, t);
    a.ring1[d][idx] = make_uint4(0u, 0u, 0u, 0u);
  } else if (bid < a.first_map) {
    copies_body<float>(a.copies, bid - a.first_pad, a.first_h0 - a.first_pad, tid);
  } else {
    frame_map_body(bid - a.first_map, a.lens, a.T, a.B, a.fidx, a.count);
  }
}
std::mutex g_capacity_mu;
std::map<std::pair<int, const void*>, int> g_capacity;    // (device, kernel) -> work-groups of the kernel that device holds at once

// How many work-groups of `kernel` the current device holds at once, one per compute unit (0 if that cannot be found out).
template <typename K>
int capacity(K kernel) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return 0; }
  std::lock_guard<std::mutex> lock(g_capacity_mu);
  const auto key = std::make_pair(dev, (const void*)kernel);
  auto it = g_capacity.find(key);
  if (it == g_capacity.end()) {
    int per_cu = 0;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    it = g_capacity.emplace(key, std::min(per_cu, 1) * prop.multiProcessorCount).first;
  }
  return it->second;
}

}  // namespace
int device_capacity(const void* kernel) { return capacity(kernel); }
namespace {

// Cooperative launches over the batch in slabs of whole 16-row tiles (or of all rows).  A work-group owns `rows_per_group` rows
// (16 or 8), so a row group takes ntile * ndir work-groups; as many row groups as the device can hold at
// once go into one launch (the kernels need every work-group of a launch resident together), the rest follow in
// further launches on the same stream: batch rows never interact, each launch walks all T steps of its rows.
// Between launches the table in which exchange groups record their XCD is cleared again.  Returns
// hipErrorCooperativeLaunchTooLarge without launching anything if not even one row tile fits.
// Return values: hipSuccess; hipErrorCooperativeLaunchTooLarge = NOTHING was launched (the caller may use another
// kernel form or the per-step path on the untouched state); any other error = a later slab failed after earlier
// slabs had already advanced the state of their rows, so the call as a whole has failed and nothing may be re-run.
template <typename K, typename A>
hipError_t coop_slabs(K kernel, int ntile, int rows_per_group, const A& a, hipStream_t s, int nrow = 0) {
  const int per_rt = rows_per_group > 16 ? 1 : 16 / rows_per_group;
  if (nrow == 0) nrow = cdiv(a.B, rows_per_group);
  const long cap = capacity(kernel);
  const long most = cap / ((long)ntile * a.ndir);                      // row groups per launch
  const int slab = most >= nrow ? nrow : (int)(most / per_rt * per_rt);
  if (slab < 1) return hipErrorCooperativeLaunchTooLarge;
  for (int row0 = 0; row0 < nrow; row0 += slab) {
    A copy = a;
    copy.rt0 = row0 / per_rt;
    copy.slab0 = row0; copy.slab_tiles = rows_per_group / 16;          // (the float kernels)
    copy.map.ntile = ntile;
    copy.map.nrow = std::min(slab, nrow - row0);
    const int groups = copy.map.nrow * a.ndir, gpx = cdiv(groups, 8);
    copy.map.gpx = (long)gpx * ntile <= cap / 8 ? gpx : 0;
    const dim3 grid(copy.map.gpx ? 8 * gpx * ntile : groups * ntile);
    if (row0 > 0 && a.xcc) {
      const hipError_t e = launch_fill_zero(a.xcc, (size_t)ntile * slab * a.ndir * 4, s);
      if (e != hipSuccess) return e == hipErrorCooperativeLaunchTooLarge ? hipErrorLaunchFailure : e;
    }
    void* args[] = {&copy};
    // (the grid has been checked against what the device holds at once either way; a cooperative launch goes through a
    // queue of its own, and crossing to it and back leaves the device idle for tens of microseconds)
    const hipError_t e = a.plain_launch ? hipLaunchKernel((const void*)kernel, grid, dim3(256), args, 0, s)
                                        : hipLaunchCooperativeKernel((const void*)kernel, grid, dim3(256), args, 0, s);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      if (row0 == 0) return hipErrorCooperativeLaunchTooLarge;         // the first launch was refused: nothing has run
      return e == hipErrorCooperativeLaunchTooLarge ? hipErrorLaunchFailure : e;
    }
  }
  return hipSuccess;
}
// The kernels address a frame's arrays with 32-bit byte offsets and park idle lanes at offset 0x7ff00000: every frame
// array (gate pre-activations [B][4n] float, outputs [B][ld] bf16) and every ring must end below that offset.
inline bool offsets_fit(long B, long n, long ld_out, long ring_bytes) {
  const long lim = 0x7ff00000L;
  return B * 4 * n * 4 < lim && B * ld_out * 2 < lim && ring_bytes < lim;
}
template <typename K>
bool slab_fits(K kernel, int ntile, int rows_per_group, int nrow, int ndir) {
  return capacity(kernel) >= (long)ntile * std::min(16 / rows_per_group, nrow) * ndir;
}
// The form of a kernel for n units: as much of the registers' worth of weights, MFMAs and ring loads per step as n needs.  The 8-row kernels in quarters
// forward (us a step, 16 rows, both directions, with half / all of it and now: n = 144 0.98 / 0.90, 256 1.00 / 0.93, 563 1.33 / 1.26, 768 1.39 / 1.30; inference 0.97 / 0.88, 0.98 / 0.90,
// 1.30 / 1.20, 1.37 / 1.25); backward a quarter, a half, and from there in eighths up to three quarters (563 1.45 / 1.33, 768 1.51 / 1.41; three eighths for n = 300 1.13 / 1.13,
// seven for 850 1.55 / 1.52: not worth a form).
typedef void (*FwdKernel)(PFwdArgs);
typedef void (*BwdKernel)(PBwdArgs);
FwdKernel fwd8_for(int n) {
  switch (cdiv(n, 256)) {
    case 0: case 1: return persist_fwd8_kernel<1>;
    case 2: return persist_fwd8_kernel<2>;
    case 3: return persist_fwd8_kernel<3>;
    default: return persist_fwd8_kernel<4>;
  }
}
FwdKernel fwd8_rows_w_for(int n) {
  switch (cdiv(n, 256)) {
    case 0: case 1: return persist_fwd8_rows_w_kernel<1>;
    case 2: return persist_fwd8_rows_w_kernel<2>;
    case 3: return persist_fwd8_rows_w_kernel<3>;
    default: return persist_fwd8_rows_w_kernel<4>;
  }
}
FwdKernel fwd16_for(int n) { return n <= 512 ? persist_fwd16r_kernel<4> : persist_fwd16r_kernel<8>; }
BwdKernel bwd8_for(int n) {
  switch (bwdp8_nct(n)) {
    case 4: return persist_bwdp_kernel<4, 4>;
    case 8: return persist_bwdp_kernel<4, 8>;
    case 10: return persist_bwdp_kernel<6, 10>;
    case 12: return persist_bwdp_kernel<6, 12>;
    default: return persist_bwdp_kernel<8, 16>;
  }
}
BwdKernel bwd16_for(int n) { return n <= 256 ? persist_bwdp16_kernel<4, 4> : n <= 512 ? persist_bwdp16_kernel<4, 8> : persist_bwdp16_kernel<8, 16>; }

}  // namespace

// More rows than the 8-row form holds in one launch go to the 16-row form, if that takes a single launch.
int persist_fwd_rows(int B, int n, int ndir) {
  const long t32 = cdiv(n, 32);
  return t32 * cdiv(B, 8) * ndir > capacity(fwd8_for(n)) && t32 * cdiv(B, 16) * ndir <= capacity(fwd16_for(n)) ? 16 : 8;
}
// W_h as it lies in memory (8 rows a group): where one launch holds the batch.  Not packing saves once, every further launch starts later (inference,
// us, packed / as it lies; n = 1000, both directions: one launch 74 / 69, three 147 / 145, six 243 / 243; n = 1024: 74 / 71, 143 / 146, 243 / 255; n = 760,
// one direction: 56 / 54, three launches 114 / 118, six 199 / 211; n = 520, both: 64 / 61, 179 / 184, 233 / 242).  Longer sequences, 34 steps: n = 1024, one direction, four launches
// 339 / 356, n = 904 327 / 331, n = 664 433 / 430, but n = 760 441 / 424 and, in three, n = 664 328 / 320: with three loads a step the other's order of chunks makes steps
// 0.1 us shorter there, but not in both directions at n = 760 (241 / 242).
bool persist_fwd_w_rows(int B, int n, int ndir) { return n % 8 == 0 && (long)cdiv(n, 32) * cdiv(B, 8) * ndir <= capacity(fwd8_rows_w_for(n)); }
int persist_bwd_rows(int B, int n, int ndir) {
  const long t32 = cdiv(n, 32);
  return t32 * cdiv(B, 8) * ndir > capacity(bwd8_for(n)) && t32 * cdiv(B, 16) * ndir <= capacity(bwd16_for(n)) ? 16 : 8;
}
// Row places of a launch that may take rows of different lengths one behind the other; 0: not this batch.  Batches that one launch of the
// 8-row kernels holds have nothing to gain (for n <= 512 that is 128 rows at least); with this, the others are those of a single
// launch of the 16-row kernels, which the lengths choose from (rows_pay).
int persist_pack_slots(int T, int B, int n, int ndir, bool backward) {
  if (n <= 512 || n > 1024 || B > kPackMaxRows || (long)T * B * n * 16 >= 0x7ff00000L) return 0;
  if ((backward ? persist_bwd_rows(B, n, ndir) : persist_fwd_rows(B, n, ndir)) != 16) return 0;
  const long per_group = (long)cdiv(n, 32) * ndir;
  const int groups = (int)std::min((backward ? capacity(persist_bwd_rows_kernel) : capacity(persist_fwd_rows_kernel)) / per_group, (long)kPackMaxSlots / 8);
  return groups < cdiv(B, 8) && groups >= cdiv(B, 16) ? groups * 8 : 0;
}
// Longest table that still pays, against T steps of the 16-row kernels.  n = 1000, 64 rows of 300 frames, both directions, start-up included:
// forward 777 us there, 863 for 600 steps here (line at 1.75 T with the padded frames' fill); backward 760 and 982 (1.53 T).  Rows of 30 to
// 300 frames, a table of 330 steps: 711 and 720 us there, 508 and 557 here.
int pack_max_steps(int T, bool backward) { return (int)((long)T * (backward ? 24 : 27) / 16); }
int pack_tab_steps(int T, int B, int slots) { return (int)((long)T * B / slots) + T + 1; }      // (fewest frames so far: at most the average, and the row's own)
hipError_t launch_fill_padded(const int* lens, const int* steps, int T, int B, int n, int ndir, void* y, float* const* cs, const float* const* c0, const int* rev, hipStream_t s) {
  const auto a16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  FillArgs a = {lens, steps, T, B, n, ndir, (uint16_t*)y, {cs[0], cs[1]}, {c0[0], c0[1]}, {rev[0], rev[1]}, 0, 0};
  a.vec_y = a16(y) && (long)ndir * n % 8 == 0;
  a.vec_c = n % 4 == 0 && a16(cs[0]) && a16(cs[1]) && a16(c0[0]) && a16(c0[1]);
  hipLaunchKernelGGL(fill_padded_kernel, dim3(B, cdiv(T, 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_persist_fwd(const PFwdArgs& a, hipStream_t s) {
  if (!persist_fwd_fits(a)) return hipErrorCooperativeLaunchTooLarge;
  if (a.slots > 0) return coop_slabs(persist_fwd_rows_kernel, cdiv(a.n, 32), 8, a, s, a.slots / 8);
  const int rows = persist_fwd_rows(a.B, a.n, a.ndir);
  return coop_slabs(rows == 16 ? fwd16_for(a.n) : a.w_rows ? fwd8_rows_w_for(a.n) : fwd8_for(a.n), cdiv(a.n, 32), rows, a, s);
}
// Would launch_persist_fwd launch anything?  (Asked before the initial state's term is added to the pre-activations,
// which only the single-launch kernels expect there.)
bool persist_fwd_fits(const PFwdArgs& a) {
  if (a.nkc > kLLMaxNkcFwd) return false;
  if (!offsets_fit(a.B, a.n, std::max(a.d[0].ldy, a.d[a.ndir - 1].ldy), (long)cdiv(a.B, 16) * a.nkc * 1024)) return false;
  return slab_fits(a.w_rows ? fwd8_rows_w_for(a.n) : fwd8_for(a.n), cdiv(a.n, 32), 8, cdiv(a.B, 8), a.ndir);
}
bool persist_bwd_fits(const PBwdArgs& a) {
  if (!offsets_fit(a.B, a.n, std::max(a.d[0].lddy, a.d[a.ndir - 1].lddy), (long)bwdp_ring_bytes(a.B, a.n))) return false;
  return a.n <= 1024 && slab_fits(bwd8_for(a.n), cdiv(a.n, 32), 8, cdiv(a.B, 8), a.ndir);
}
hipError_t launch_persist_bwd(const PBwdArgs& a, hipStream_t s) {
  if (a.slots > 0) return coop_slabs(persist_bwd_rows_kernel, cdiv(a.n, 32), 8, a, s, a.slots / 8);
  const int rows = persist_bwd_rows(a.B, a.n, a.ndir);
  return coop_slabs(rows == 16 ? bwd16_for(a.n) : bwd8_for(a.n), cdiv(a.n, 32), rows, a, s);
}
static int pad_blocks(const SetUpCopies& c) { return c.x ? cdiv(c.x_rows * (c.x_ld / 8), 256) : 0; }
static int h0_blocks(const SetUpCopies& c) { return c.h0 ? cdiv((long)c.ndir * c.B * c.ld, 256) : 0; }
hipError_t launch_prep_fwd_ll(const ZeroRegions& z, const void* W, uint4* Wf, int n, int nkc, int ndir, bool paired, uint4* ring0, uint4* ring1,
                              int nrt, const FrameMapArgs& fm, const PackRows& rows, const SetUpCopies& copies, const GemmArgs* zx, hipStream_t s) {
  if (z.overflow) return hipErrorInvalidValue;
  PrepArgs a = {};
  a.z = z; a.W = (const bf16_t*)W; a.Wout = Wf; a.n = n; a.paired = paired; a.nk = nkc;
  a.w_total = Wf ? (long)(ndir * ll_wf_bytes(n, nkc) / 16) : (long)ndir * n * n * 2;       // chunks, or dwords to fetch
  a.ring0 = ring0; a.ring1 = ring1; a.ring_total = (long)ndir * nrt * nkc * 64 * 2;
  a.first_pack = z.count ? z.first_block[z.count] : 0;
  a.first_ring = a.first_pack + (int)cdiv(a.w_total, Wf ? 256 : 256 * 16 * kTouch);
  a.copies = copies;
  a.first_pad = a.first_ring + cdiv(a.ring_total, 256);
  a.first_h0 = a.first_pad + pad_blocks(copies);
  a.first_map = a.first_h0 + h0_blocks(copies);
  a.backward = 0;
  a.lens = fm.lens; a.T = fm.T; a.B = fm.B; a.fidx = fm.fidx; a.count = fm.count;
  a.rows = rows;
  if (zx) {
    const GemmArgs& g = *zx;
    FewZxArgs f = {(const uint16_t*)g.A, (const uint16_t*)g.B, g.bias, (float*)g.C, g.M, g.K, g.N, cdiv(g.N, 16 * kFewUnits), g.nz, cdiv(g.N, 16 * kFewUnits) * g.nz * cdiv(g.M, 64), g.sCz};
    const dim3 grid(f.blocks + cdiv(a.first_map, 2)), block(512);
    if (g.M <= 16) hipLaunchKernelGGL(prep_zx_kernel<1>, grid, block, 0, s, a, f);
    else if (g.M <= 32) hipLaunchKernelGGL(prep_zx_kernel<2>, grid, block, 0, s, a, f);
    else hipLaunchKernelGGL(prep_zx_kernel<4>, grid, block, 0, s, a, f);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(prep_ll_kernel, dim3(a.first_map + (fm.fidx ? cdiv(fm.T, 4) : 0) + (rows.slots > 0 ? 1 : 0)), dim3(256), 0, s, a);
  return hipGetLastError();
}
// g: the input projection, from the caller's arrays.  x by 16 bytes that begin at any whole word, W_x by words, results by 16 bytes.
bool few_zx_ok(const GemmArgs& g) {
  const long rounds = cdiv((long)cdiv(g.N, 16 * kFewUnits) * g.nz * cdiv(g.M, 64), 256);
  return g.in_bf16 && !g.out_bf16 && g.M > 0 && g.M <= kFewZxRows && rounds * g.K <= kFewZxWalk && rounds <= (g.K % 8 == 0 ? 5 : 6) &&
         g.K % 2 == 0 && g.N % 4 == 0 && g.lda == g.K && g.ldb == g.N && g.ldc == g.N && g.sBz == (long)g.K * g.N && g.sCz % 4 == 0 && (long)(g.K + 1024) * g.N * 2 < 0x7ff00000L;
}
hipError_t launch_prep_bwd_ll(const ZeroRegions& z, const void* W, uint4* Wb, int n, int ndir, bool paired, int nct, const FrameMapArgs& fm, const PackRows& rows, const SetUpCopies& copies, hipStream_t s) {
  if (z.overflow) return hipErrorInvalidValue;
  PrepArgs a = {};
  a.z = z; a.W = (const bf16_t*)W; a.Wout = Wb; a.n = n; a.nk = cdiv(n, 32); a.nct = nct; a.w_total = (long)ndir * a.nk * 4 * 4 * a.nct * 64;
  a.first_pack = z.count ? z.first_block[z.count] : 0;
  a.first_ring = a.first_pack + cdiv(a.w_total, 256);
  a.copies = copies;
  a.first_pad = a.first_ring;
  a.first_h0 = a.first_map = a.first_pad + pad_blocks(copies);
  a.backward = 1; a.paired = paired;
  a.lens = fm.lens; a.T = fm.T; a.B = fm.B; a.fidx = fm.fidx; a.count = fm.count;
  a.rows = rows;
  hipLaunchKernelGGL(prep_ll_kernel, dim3(a.first_map + (fm.fidx ? cdiv(fm.T, 4) : 0) + (rows.slots > 0 ? 1 : 0)), dim3(256), 0, s, a);
  return hipGetLastError();
}
// The float kernels' form for n units: as many chunks of h (forward) and column tiles (backward) to a wavefront as n needs, in twos, since a form's products, ring loads and
// published blocks are the same whatever n it is used for.  us a step, forward and backward, 27 rows, both directions, in the next power of two's form / its own: n = 300 2.61 3.73 / 2.30
// 3.22, 563 4.32 5.61 / 3.37 4.37, 700 4.44 5.67 / 3.75 4.97, 850 4.62 6.02 / 4.30 5.93; 64 rows of 563 7.50 8.39 / 5.62 7.65.  (Up to 512 the exchange is inside an XCD.)
FwdKernel fwd_f32_for(int n) {
  switch (cdiv(n, 128)) {
    case 0: case 1: case 2: return persist_fwd_f32_kernel<4>;
    case 3: return persist_fwd_f32_kernel<6>;
    case 4: return persist_fwd_f32_kernel<8>;
    case 5: return persist_fwd_f32_kernel<10>;
    case 6: return persist_fwd_f32_kernel<12>;
    case 7: return persist_fwd_f32_kernel<14>;
    default: return persist_fwd_f32_kernel<16>;
  }
}
BwdKernel bwd_f32_for(int n) {
  switch (bwd_f32_nct(n)) {
    case 4: return persist_bwd_f32_kernel<4>;
    case 6: return persist_bwd_f32_kernel<6>;
    case 8: return persist_bwd_f32_kernel<8>;
    case 10: return persist_bwd_f32_kernel<10>;
    case 12: return persist_bwd_f32_kernel<12>;
    case 14: return persist_bwd_f32_kernel<14>;
    default: return persist_bwd_f32_kernel<16>;
  }
}
// A work-group is one row tile where the device holds all of them so, else two.
template <typename K>
int f32_rows_per_group(K kernel, int ntile, int B, int ndir) { return (long)ntile * cdiv(B, 16) * ndir <= capacity(kernel) ? 16 : 32; }

// Few steps, or batches that take several launches, are faster in the per-step kernels (n = 700, 300 rows, both directions, 20 steps: forward
// 1387 us here, 838 there).  Both sides as they were measured, in us, for n from 130 to 1024, 1 to 512 rows, 2 to 60 steps, one and two
// directions, plain and cooperative launches (1573 shapes): the choice was within 5 % of the faster side in 99 % of them and never 1.25 times
// it; always the loops was up to 2.8 times the other.  The loops' side has been measured again since their products are bfloat16 parts (4 and 100 steps of 11
// shapes): of 396 shapes of 2 to 24 steps the choice is within 5 % of the per-step kernels or faster in 95 %, never 1.16 times them.  With lengths given, a pair of row tiles is taken to have work for 0.8 of its steps.
// Both sides have become faster since (a form for every 128 units and a set-up of one launch here, more wavefronts there), and the line has not moved with them: the loops carry sums of
// 2^32 and more with 16 significant bits and add in the order of arrival, the per-step kernels keep 24 bits and repeat theirs, and no call is to lose that for a faster kernel.
// A line by the present times gives the loops some calls more (us, per step / here: forward and backward of 4 steps of 2 rows, n = 700, both directions, ordinary launches 85 / 51 and 156 / 92).
bool persist_f32_pays(int T, int B, int n, int ndir, bool lens, bool plain_launch, bool backward) {
  const int form = n <= 256 ? 0 : n <= 512 ? 1 : 2, ntile = cdiv(n, 16), cap = backward ? capacity(bwd_f32_for(n)) : capacity(fwd_f32_for(n));
  const bool one = (long)ntile * cdiv(B, 16) * ndir <= cap, pair = !one && B > 16;
  const int launches = one ? 1 : cdiv(cdiv(B, 32), std::max(1, cap / (ntile * ndir)));
  const double w = (double)n * n / (1024.0 * 1024.0) * ndir, nr = (double)n * ndir * B * 1e-5, nnr = nr * n * 1e-3, part = lens && pair ? 0.8 : 1.0;
  double here, there;
  if (backward) {
    const double step[2][3] = {{2.8, 4.3, 7.2}, {7.2, 9.3, 17.4}};
    here = 34.0 + 18.0 * w + launches * (plain_launch ? 30.0 : 51.0) + launches * T * step[pair][form] * part;
    there = 58.3 + 16.0 * w + T * std::max(4.25 + 17.1e-3 * n + 6.6 * nr + 10.4 * nnr, 22.0 * nnr);
  } else {
    const double step[2][3] = {{1.9, 2.65, 4.25}, {4.2, 6.2, 9.2}};
    here = 19.0 + 11.7 * w + launches * (plain_launch ? 15.0 : 36.0) + launches * T * step[pair][form] * part;
    there = 27.9 + 7.8 * w + T * std::max(3.8 + 6.15e-3 * n + 4.15 * nr + 4.9 * nnr, 10.9 * nnr);
  }
  return here < there;
}
bool persist_fwd_f32_fits(const PFwdArgs& a) {
  if (a.n > 1024 || a.T < 2) return false;
  const long ring_bytes = (long)cdiv(a.B, 16) * a.nkc * 1024;
  return ring_bytes < 0x7ff00000L && (long)cdiv(a.n, 16) * a.ndir <= capacity(fwd_f32_for(a.n));
}
hipError_t launch_persist_fwd_f32(const PFwdArgs& a, hipStream_t s) {
  if (!persist_fwd_f32_fits(a)) return hipErrorCooperativeLaunchTooLarge;
  const auto kernel = fwd_f32_for(a.n);
  return coop_slabs(kernel, cdiv(a.n, 16), f32_rows_per_group(kernel, cdiv(a.n, 16), a.B, a.ndir), a, s);
}
bool persist_bwd_f32_fits(const PBwdArgs& a) {
  if (a.n > 1024 || a.T < 2) return false;
  const long ntile = cdiv(a.n, 16);
  if ((long)cdiv(a.B, 16) * ntile * ntile * 1024 >= 0x7ff00000L) return false;
  return ntile * a.ndir <= capacity(bwd_f32_for(a.n));
}
static hipError_t prep_f32(PrepF32Args a, const ZeroRegions& z, int ndir, const FrameMapArgs& fm, const SetUpCopies& copies, hipStream_t s) {
  if (z.overflow) return hipErrorInvalidValue;
  a.z = z;
  a.first_pack = z.count ? z.first_block[z.count] : 0;
  a.first_ring = a.first_pack + cdiv(a.w_total, 256);
  a.per_ring = cdiv(a.ring_total, 256);
  a.copies = copies;
  a.first_pad = a.first_ring + ndir * a.per_ring;
  a.first_h0 = a.first_pad + pad_blocks(copies);
  a.first_map = a.first_h0 + h0_blocks(copies);
  a.lens = fm.lens; a.T = fm.T; a.B = fm.B; a.fidx = fm.fidx; a.count = fm.count;
  hipLaunchKernelGGL(prep_f32_kernel, dim3(a.first_map + (fm.fidx ? cdiv(fm.T, 4) : 0)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_prep_fwd_f32(const ZeroRegions& z, const void* W, void* Wf, const PFwdArgs& p, const FrameMapArgs& fm, const SetUpCopies& copies, hipStream_t s) {
  PrepF32Args a = {};
  a.W = (const float*)W; a.Wout = Wf; a.n = p.n; a.nk = p.nkc; a.w_total = (long)p.ndir * cdiv(p.n, 8) * 2 * p.nkc * 64;
  for (int d = 0; d < p.ndir; ++d) { a.ring0[d] = p.d[d].ring0; a.ring1[d] = p.d[d].ring1; }
  a.ring_total = (long)cdiv(p.B, 16) * p.nkc * 64;
  return prep_f32(a, z, p.ndir, fm, copies, s);
}
hipError_t launch_prep_bwd_f32(const ZeroRegions& z, const void* W, void* Wb, int n, int ndir, const FrameMapArgs& fm, const SetUpCopies& copies, hipStream_t s) {
  PrepF32Args a = {};
  a.W = (const float*)W; a.Wout = Wb; a.n = n; a.nk = cdiv(n, 16); a.nct = bwd_f32_nct(n); a.w_total = (long)ndir * a.nk * 4 * a.nct * 64;
  a.backward = 1;
  return prep_f32(a, z, ndir, fm, copies, s);
}
// (the rings must hold zeros)
hipError_t launch_persist_bwd_f32(const PBwdArgs& a, hipStream_t s) {
  if (!persist_bwd_f32_fits(a)) return hipErrorCooperativeLaunchTooLarge;
  const auto kernel = bwd_f32_for(a.n);
  return coop_slabs(kernel, cdiv(a.n, 16), f32_rows_per_group(kernel, cdiv(a.n, 16), a.B, a.ndir), a, s);
}
}  // namespace lstm
