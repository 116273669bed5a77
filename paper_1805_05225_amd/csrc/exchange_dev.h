// Device helpers of the kernels whose work-groups exchange data inside a launch.
#pragma once
#include "recurrent_dev.h"

namespace lstm {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
constexpr int kBufFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9-family devices
// cache policy of the polling loads: bit 4 = coherent at agent scope (bypasses the XCD-local L2),
// bit 31 = volatile, so the compiler re-issues the load in every poll
constexpr int kSc1 = (int)(16u | 0x80000000u);

// Floats that travel with a tag in bit 30 (partial sums scaled by 2^-32).  Below 1 in magnitude - 2^32 before the scaling - that
// bit is 0 and the value travels as it is.  Anything else, infinities and NaN included, is folded into the patterns between 1 and 2:
// sign, exponent and 15 bits of the mantissa, rounded.  One bit pattern either way, so value and tag still arrive together.  Exactly
// 1 is no value: it says that the folded one follows (a writer that looks for wide values only after it has published).
constexpr unsigned kOneBits = 0x3f800000u, kInfBits = 0x7f800000u;
__host__ __device__ constexpr unsigned fold_wide(unsigned v) {
  const unsigned m = v & 0x7fffffffu;
  if (m < kOneBits) return v;
  const unsigned t = m > kInfBits ? 0x40400000u : m - kOneBits + 0x80u;          // (every NaN: the quiet one)
  return (v & 0x80000000u) | (kOneBits + 1u + (t >> 8));
}
__host__ __device__ constexpr unsigned unfold_wide(unsigned v) {
  const unsigned m = v & 0x7fffffffu;
  return m <= kOneBits ? v : (v & 0x80000000u) | (((m - kOneBits - 1u) << 8) + kOneBits);
}
static_assert(unfold_wide(fold_wide(0x3f7fffffu)) == 0x3f7fffffu && unfold_wide(fold_wide(0xbf800000u)) == 0xbf800000u, "in range, and 1");
static_assert(unfold_wide(fold_wide(kInfBits)) == kInfBits && unfold_wide(fold_wide(0xff800000u)) == 0xff800000u, "infinities");
static_assert(unfold_wide(fold_wide(0x7fffffffu)) > kInfBits && unfold_wide(fold_wide(0x7f800001u)) > kInfBits, "NaN");
static_assert(unfold_wide(fold_wide(0x6f12347fu)) == 0x6f123400u && unfold_wide(fold_wide(0xef123480u)) == 0xef123500u, "16 bits, rounded");
static_assert(fold_wide(0x7fffffffu) < 0x40000000u && fold_wide(0x7f7fffffu) < 0x40000000u && fold_wide(kOneBits) > kOneBits, "bit 30 is free, 1 is none");
// the largest of m and the magnitudes of two floats; NaN if one of them is
__device__ __forceinline__ float max_magnitude(float m, float a, float b) {
  asm("v_maximum3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(a), "v"(b));
  return m;
}
__device__ __forceinline__ bool is_wide(float m) { return !(m < 1.f); }        // of a magnitude

__device__ __forceinline__ unsigned ld_relaxed(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Is every work-group of this one's exchange group on the same XCD?  Then their ring stores need not be written
// through to memory: the XCD's L2 is the point where those work-groups meet (measured: one-way latency 212 ns
// instead of 350, and the ring's store traffic stays out of the fabric).  Each work-group publishes the XCD it runs on
// (hardware register XCC_ID) in `tab` (zero-filled by the host, one word per work-group, a group's words consecutive
// from `group_base`) and reads the group's words; anything but "all equal to mine" - a word still unset after the
// poll limit included - means "not local", and the caller then uses agent-scope stores as before.  The verdict
// needs no agreement: a work-group that says "local" has seen every member on its own XCD.
// The words are published before W_h is loaded and looked at behind it, a lane per member (one thread reading 32 words
// one after the other held every launch up by 10 us).
__device__ __forceinline__ unsigned my_xcd() { return (__builtin_amdgcn_s_getreg(((4 - 1) << 11) | 20) & 15u) + 1u; }   // XCC_ID, bits 3:0
__device__ __forceinline__ void publish_xcd(unsigned* tab, int group_base, int me) {
  if (tab && threadIdx.x == 0) st_relaxed(&tab[group_base + me], my_xcd());
}
__device__ __forceinline__ int group_is_xcd_local(unsigned* tab, int group_base, int members, unsigned limit) {
  __shared__ int verdict;
  if (threadIdx.x < 64) {
    const unsigned mine = my_xcd();
    bool same = tab != nullptr;
    for (int p = threadIdx.x; p < members && same; p += 64) {
      unsigned v = 0u;
      for (unsigned poll = 0; poll < limit; ++poll) {
        v = ld_relaxed(&tab[group_base + p]);
        if (v != 0u) break;
      }
      same = v == mine;
    }
    const bool all = __builtin_amdgcn_ballot_w64(!same) == 0ull;
    if (threadIdx.x == 0) verdict = all ? 1 : 0;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(verdict);
}

}  // namespace
}  // namespace lstm
