// One step of batched beam search on the device (Sec. 3, Table 2: decoding is a batched beam search that runs on the GPU, beam
// size 12; Listing 1: "output_prob" softmax over the labels, "output" chooses, "trg" embeds the choice):
//
//     cand[q, b, v] = score[q, b] + logits[r, v] - logsumexp(logits[r, :]),  r = q * beam + b
//     the `beam` largest candidates of sentence q, best first, equal ones by ascending b * V + v  -> score', src, label
//     state rows follow their hypotheses: out[q * beam + k] = in[q * beam + src[q, k]]
//     trg[r] = W_trg[label[r]] + b_trg
//
// No candidate list of beam * V entries is ever sorted: a sentence's best `beam` candidates contain at most `beam` from one
// row, so every row first picks its own best `beam` labels in one pass over its logits (beam_row_kernel, a work-group per row
// or, of few rows, per stretch of one), and a work-group per sentence merges the survivors (beam_merge_kernel).  Nothing
// returns to the host.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "../../include/lstm_abi.h"
#include "common.h"
#include "exchange_dev.h"

namespace lstm {
namespace {

constexpr int kBeamMax = 16;
constexpr int kVocabMax = 1 << 26;    // beam * V must fit an int32 flat index
constexpr int kRowPieces = 24;        // 16-byte pieces of a row that a thread holds at most
constexpr int kRowParts = 8;          // stretches of a row at most
constexpr long kRowGroups = 768;      // work-groups up to which rows are cut into stretches

// Scratch of lstm_beam_step_static: Q * beam * beam survivors (value and label) at most kStaticCands of each, e.g. 256
// sentences at beam 16.  512 KiB of every device the library runs on, held until the process ends.
constexpr uint64_t kStaticCands = 1u << 16;
constexpr int kStaticDevices = 64;
static __device__ __align__(256) unsigned char scratch[2 * kStaticCands * 4];
std::mutex g_static_mu;
void* g_static_ptr[kStaticDevices] = {};   // device address of `scratch` per device, from hipGetSymbolAddress

// (value, index) pairs ordered by larger value first, then smaller index: `better(a, b)` = a comes before b
struct Cand { float v; int i; };
__device__ __forceinline__ bool better(const Cand& a, const Cand& b) { return (a.v > b.v) | ((a.v == b.v) & (a.i < b.i)); }
// field by field: selecting between two structs made the compiler store both to scratch memory and load one back
__device__ __forceinline__ Cand pick(const Cand& a, const Cand& b) {
  const bool t = better(a, b);
  Cand c;
  c.v = t ? a.v : b.v;
  c.i = t ? a.i : b.i;
  return c;
}
// The best candidate of the wavefront, in every lane.  Six combining steps through DPP moves (neighbour in the quad, other
// pair of the quad, mirrored half row, mirrored row, last lane of the row before, last lane of the first half), after
// which lane 63 holds the result; 64 lanes of `__shfl_xor` took six dependent trips through the LDS crossbar per value.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ Cand dpp_step(const Cand& c) {
  Cand d;   // lanes that the move does not reach (row mask, row_bcast sources out of range) keep their own candidate
  d.v = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(c.v), __float_as_int(c.v), CTRL, ROW_MASK, 0xf, false));
  d.i = __builtin_amdgcn_update_dpp(c.i, c.i, CTRL, ROW_MASK, 0xf, false);
  return pick(c, d);
}
__device__ __forceinline__ Cand wave_best(Cand c) {
  c = dpp_step<0xB1, 0xf>(c);       // quad_perm [1,0,3,2]
  c = dpp_step<0x4E, 0xf>(c);       // quad_perm [2,3,0,1]
  c = dpp_step<0x141, 0xf>(c);      // row_half_mirror
  c = dpp_step<0x140, 0xf>(c);      // row_mirror: every lane holds the best of its row of 16
  c = dpp_step<0x142, 0xa>(c);      // row_bcast15 into rows 1 and 3
  c = dpp_step<0x143, 0xc>(c);      // row_bcast31 into rows 2 and 3
  Cand w;
  w.v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c.v), 63));
  w.i = __builtin_amdgcn_readlane(c.i, 63);
  return w;
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_max(unsigned c) { return max(c, (unsigned)__builtin_amdgcn_update_dpp((int)c, (int)c, CTRL, ROW_MASK, 0xf, false)); }
__device__ __forceinline__ unsigned wave_max(unsigned c) {        // (the same steps)
  c = dpp_max<0x142, 0xa>(dpp_max<0x140, 0xf>(dpp_max<0x141, 0xf>(dpp_max<0x4E, 0xf>(dpp_max<0xB1, 0xf>(c)))));
  return (unsigned)__builtin_amdgcn_readlane((int)dpp_max<0x143, 0xc>(c), 63);
}
// The choice of a work-group's best `need` candidates, best first, out of what its NW wavefronts hold in registers.
template <int NW>
struct Chooser {
  static constexpr int kSeg = NW == 1 ? 64 : 128;                // finalists a wavefront may contribute
  unsigned key[64 * NW];
  float v[NW][kSeg], out_v[kBeamMax], win_v[NW];
  int i[NW][kSeg], out_i[kBeamMax], win_i[NW], count[NW];
};
// `top` is the largest value this thread has seen (its own entries or earlier ones that the list so far holds), each(f) calls
// f(value, index) for every entry and scan(bound, f) for every entry that is not surely below the bound; both are wavefront-wide.  -inf and NaN are no candidates.  Results in s.out_v / out_i[0 .. need), (-inf, 0x7fffffff) where there are
// fewer; the caller synchronises before the next use of s.
// An entry strictly below the need-th largest of 64 values seen (a lane's `top`s, the largest of all wavefronts') has `need` entries in front of it.  That bound is found by bisection over
// the ordered bit patterns (20 bits of them, rounded down) between the least and the largest of the 64, a ballot a step, ended where exactly `need` are above (over 256 values with four ballots a step, and
// always 20 of them, it took 0.6 us more); what reaches it - little more than `need` entries unless values
// repeat - goes to a list in LDS, a stretch per wavefront, and the place of a finalist is the number of better ones.  Lists that do not
// fit (plateaus) are left: `need` rounds of "every thread offers its best behind the last winner" over the registers take their place.
template <int NW, typename Each, typename Scan>
__device__ __forceinline__ void choose_best(Chooser<NW>& s, float top, int need, Each each, Scan scan) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float kNegInf = -__builtin_inff();
  const unsigned f = __float_as_uint(top);
  unsigned key = ((f & 0x80000000u) ? ~f : (f | 0x80000000u)) >> 12;           // larger float => key not smaller
  if constexpr (NW > 1) {
    s.key[threadIdx.x] = key;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) key = max(key, s.key[64 * w + lane]);
  }
  constexpr unsigned kNone = 0x007fffffu >> 12;                   // the key of -inf: nothing seen
  float bound = kNegInf;
  if (__popcll(__ballot(key > kNone)) >= need) {
    unsigned hi = wave_max(key), lo = ~wave_max(key > kNone ? ~key : 0u);
    while (lo < hi) {
      const unsigned mid = lo + ((hi - lo) >> 1) + 1u;
      const int n = __popcll(__ballot(key >= mid));
      if (n >= need) lo = mid; else hi = mid - 1u;
      if (n == need) break;
    }
    const unsigned full = lo << 12;                               // the smallest ordered pattern with this key
    bound = __uint_as_float((full & 0x80000000u) ? (full & 0x7fffffffu) : ~full);
  }
  int count = 0;                                                 // of this wavefront (the same in every lane)
  scan(bound, [&](float x, int idx) {
    const bool keep = x > kNegInf && x >= bound;
    const unsigned long long mask = __ballot(keep);
    if (mask == 0ull) return;
    const int pos = count + (int)__popcll(mask & ((1ull << lane) - 1ull));
    if (keep && pos < Chooser<NW>::kSeg) { s.v[wave][pos] = x; s.i[wave][pos] = idx; }
    count += (int)__popcll(mask);
  });
  if (lane == 0) s.count[wave] = count;
  if (threadIdx.x < kBeamMax) { s.out_v[threadIdx.x] = kNegInf; s.out_i[threadIdx.x] = 0x7fffffff; }
  __syncthreads();
  int most = 0, total = 0, w = 0, at = threadIdx.x;                // thread t has finalist t of the stretches, number `at` of wavefront w's
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int c = s.count[q];
    total += c;
    most = max(most, c);
    if (q + 1 < NW && (int)threadIdx.x >= total) { w = q + 1; at = threadIdx.x - total; }
  }
  if (most <= Chooser<NW>::kSeg && total <= 64 * NW) {
    const int t = threadIdx.x;
    if (wave * 64 >= total) return;
    Cand mine = {kNegInf, 0x7fffffff};
    if (t < total) { mine.v = s.v[w][at]; mine.i = s.i[w][at]; }
    int place = 0;
    if (NW == 1 || total <= 64) {
      for (int j = 0; j < total; ++j) {
        const Cand other = {__int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine.v), j)), __builtin_amdgcn_readlane(mine.i, j)};
        place += better(other, mine) ? 1 : 0;
      }
    } else {
#pragma unroll
      for (int seg = 0; seg < NW; ++seg) {
        const int n = s.count[seg];
        for (int j = 0; j < n; ++j) {
          const Cand other = {s.v[seg][j], s.i[seg][j]};
          place += better(other, mine) ? 1 : 0;
        }
      }
    }
    if (t < total && place < need) { s.out_v[place] = mine.v; s.out_i[place] = mine.i; }
    return;
  }
  Cand last = {__builtin_inff(), -1};                             // in front of every candidate
  for (int k = 0; k < need; ++k) {
    Cand mine = {kNegInf, 0x7fffffff};
    each([&](float x, int idx) {                                 // (-inf is sorted out below: a test of x alone would be kept for all rounds, in registers)
      const Cand c = {x, idx};
      if (better(last, c) && better(c, mine)) { mine.v = x; mine.i = idx; }
    });
    const Cand win = wave_best(mine);
    Cand best = win;
    if constexpr (NW > 1) {
      if (lane == 0) { s.win_v[wave] = win.v; s.win_i[wave] = win.i; }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NW; ++q) best = pick(best, Cand{s.win_v[q], s.win_i[q]});
    }
    if (threadIdx.x == 0 && best.v > kNegInf) { s.out_v[k] = best.v; s.out_i[k] = best.i; }
    last = best;
    __syncthreads();
  }
}

// What exponentials are taken relative to where the maximum may be -inf (nothing but -inf and NaN so far): exp(-inf - base) is 0 then, and a NaN stays one.
__device__ __forceinline__ float lse_base(float m) { return fmaxf(m, -__FLT_MAX__); }

// Row r of the logits in `parts` stretches, a work-group each (parts > 1: few rows, which would leave compute units
// idle): four wavefronts, or one for a row of at most 64 pieces, which four would have to meet over.  A stretch is read once, up to U loads of 16 bytes a thread in flight, and stays in registers: the logsumexp is
// folded four pieces at a time as they arrive, one bound for the whole work-group tells the few entries that can be among the best
// apart, and these are ranked (choose_best).  A stretch of more than 64 NW U pieces (of 16 bytes) takes several rounds, each with the best so far among its candidates.
// Rows start and end anywhere: 16-byte pieces between the first and the last 16-byte boundary, the up to three entries on
// either side one by one.
// What bounds it: the reading of the logits, and for few rows a round trip to memory, the bisection and the ranking behind each other.
// us a step, merge included, calls in a graph (a buffer of candidates in LDS with a bound renewed every four loads / four wavefronts for any row and a bisection over 256 values / now): 64 sentences of 12,
// V = 20000 26.4 / 20.3 / 19.2; 50 of 12, V = 20787 (rows that are not whole 16 bytes) 64.8 / 20.7 / 19.8; 8 of 13, V = 22051 48.8 / 16.7 / 14.7; 1 of 8, V = 14274 31.6 / 11.2 / 9.9; 31 of 9, V = 1853
// 12.7 / 10.8 / 9.1; 32 of 8, V = 1000 9.6 / 9.5 / 7.9; 16 of 4, V = 100 8.1 / 8.9 / 6.7; 77 of 5, V = 19 7.8 / 11.3 / 7.4.
// A NaN (or +inf) anywhere in a row makes its logsumexp and so all its scores NaN, and these never win.
// One stretch: cand_val[r][k] = score[r] + logits[r][label] - logsumexp and cand_lab[r][k].  Several: the logit itself in
// cand_val[r][part][k], and the stretch's (maximum, sum of exponentials, score) in part_sums[r][part].
template <int U, int NW>
__global__ __launch_bounds__(64 * NW) void beam_row_kernel(const float* __restrict__ logits, long ld, const float* __restrict__ score,
                                                       float* __restrict__ cand_val, int* __restrict__ cand_lab, float4* __restrict__ part_sums,
                                                       int V, int beam, int parts, int per, int step) {
  constexpr int NT = 64 * NW, G = U < 4 ? U : 4;
  __shared__ Chooser<NW> s;
  __shared__ float part_m[NW], part_z[NW];
  const int r = (int)blockIdx.x / parts, part = (int)blockIdx.x - r * parts, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* row = logits + (long)r * ld;
  const int head = min(V, (int)((4u - ((unsigned)((uintptr_t)row >> 2) & 3u)) & 3u)), n4 = (V - head) >> 2, tail = V - head - 4 * n4;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(row + head), 0, n4 * 16, kBufFlags);
  const int begin = part * per, end = min(n4, begin + per);
  const float kNegInf = -__builtin_inff();
  float m = kNegInf, z = 0.f;                                    // running maximum and sum of exp(x - m) of this thread's entries
  // an entry outside the pieces: first the row's own, later one of the best so far
  float ex = kNegInf;
  int ei = 0x7fffffff;
  if (part == 0 && tid < head + tail) {
    ei = tid < head ? tid : head + 4 * n4 + tid - head;
    ex = row[ei];
    m = fmaxf(ex, kNegInf);
    z = __expf(ex - lse_base(ex));
  }
  int base = begin;
  for (;;) {
    const int stop = min(end, base + step);
    u32x4 x4[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x4[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)(base + u * NT + tid) * 16u, 0, 0);
    float x[U][4];
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += G) {
      float mn = m;
#pragma unroll
      for (int u = u0; u < u0 + G; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[u][e] = __uint_as_float(x4[u][e]);
      if (base + (u0 + G) * NT > stop) {
        const int left = stop - base - tid;
#pragma unroll
        for (int u = u0; u < u0 + G; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) x[u][e] = u * NT < left ? x[u][e] : kNegInf;
      }
#pragma unroll
      for (int u = u0; u < u0 + G; ++u) mn = fmaxf(mn, fmaxf(fmaxf(x[u][0], x[u][1]), fmaxf(x[u][2], x[u][3])));
      if (mn > kNegInf) {
        z *= __expf(m - mn);
#pragma unroll
        for (int u = u0; u < u0 + G; ++u) z += (__expf(x[u][0] - mn) + __expf(x[u][1] - mn)) + (__expf(x[u][2] - mn) + __expf(x[u][3] - mn));
      } else {                                                   // nothing but -inf and NaN so far
#pragma unroll
        for (int u = u0; u < u0 + G; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) z = x[u][e] == kNegInf ? z : __builtin_nanf("");
      }
      m = mn;
    }
    const int first = head + 4 * (base + tid);
    const auto each = [&](auto f) {
      int i = first;
      asm volatile("" : "+v"(i));                                // (or 4 U labels are kept in registers for the rounds behind a full list)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) f(x[u][e], i + 4 * NT * u + e);
      f(ex, ei);
    };
    const auto scan = [&](float bound, auto f) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (__ballot(fmaxf(fmaxf(x[u][0], x[u][1]), fmaxf(x[u][2], x[u][3])) >= bound) == 0ull) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) f(x[u][e], first + 4 * NT * u + e);
      }
      f(ex, ei);
    };
    choose_best(s, m, beam, each, scan);
    base += step;
    if (base >= end) break;
    __syncthreads();
    ex = tid < beam ? s.out_v[tid] : kNegInf;
    ei = tid < beam ? s.out_i[tid] : 0x7fffffff;
    __syncthreads();
  }
  // logsumexp of the wavefronts' parts, then of all
  float mw = m;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mw = fmaxf(mw, __shfl_xor(mw, o));
  float zw = z * __expf(lse_base(m) - lse_base(mw));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) zw += __shfl_xor(zw, o);
  if (lane == 0) { part_m[wave] = mw; part_z[wave] = zw; }
  __syncthreads();
  if (tid >= 64) return;
  float mr = kNegInf, zr = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) mr = fmaxf(mr, part_m[w]);
#pragma unroll
  for (int w = 0; w < NW; ++w) zr += part_z[w] * __expf(lse_base(part_m[w]) - lse_base(mr));
  const float sc = score[r];
  if (parts > 1 && tid == 0) part_sums[blockIdx.x] = make_float4(mr, zr, sc, 0.f);
  if (tid < beam) {
    const bool found = s.out_i[tid] != 0x7fffffff;               // fewer than `beam` usable labels: the rest never wins
    const float v = s.out_v[tid];
    cand_val[(long)blockIdx.x * beam + tid] = !found ? kNegInf : parts > 1 ? v : sc + (v - (mr + __logf(zr)));
    cand_lab[(long)blockIdx.x * beam + tid] = found ? s.out_i[tid] : 0;
  }
}

// The beam * parts * beam survivors of sentence q = blockIdx.x: the best `beam`, by value and then by flat index b * V + label.
// 64 NW N >= that many.  One wavefront up to 256 of them: nothing to meet over.
template <int N, int NW>
__global__ __launch_bounds__(64 * NW) void beam_merge_kernel(const float* __restrict__ cand_val, const int* __restrict__ cand_lab,
                                                         const float4* __restrict__ part_sums, float* __restrict__ score_out,
                                                         int* __restrict__ src_out, int* __restrict__ label_out, int V, int beam, int parts) {
  __shared__ Chooser<NW> s;
  __shared__ float row_sc[kBeamMax], row_lse[kBeamMax];
  const int q = blockIdx.x, tid = threadIdx.x, per_row = parts * beam, total = beam * per_row;
  const float kNegInf = -__builtin_inff();
  float v[N];
  int flat[N], b[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int c = tid + 64 * NW * k;
    b[k] = c / per_row;
    v[k] = c < total ? cand_val[(long)q * total + c] : kNegInf;
    flat[k] = c < total ? b[k] * V + cand_lab[(long)q * total + c] : 0x7fffffff;
  }
  if (parts > 1) {
    if (tid < beam) {
      const float4* ps = part_sums + ((long)q * beam + tid) * parts;
      float mr = kNegInf, zr = 0.f;
      for (int p = 0; p < parts; ++p) mr = fmaxf(mr, ps[p].x);
      for (int p = 0; p < parts; ++p) zr += ps[p].y * __expf(lse_base(ps[p].x) - lse_base(mr));
      row_sc[tid] = ps[0].z;
      row_lse[tid] = mr + __logf(zr);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (v[k] > kNegInf) v[k] = row_sc[b[k]] + (v[k] - row_lse[b[k]]);
  }
  float top = kNegInf;
#pragma unroll
  for (int k = 0; k < N; ++k) top = fmaxf(top, v[k]);
  const auto each = [&](auto f) {
#pragma unroll
    for (int k = 0; k < N; ++k) f(v[k], flat[k]);
  };
  choose_best(s, top, beam, each, [&](float, auto f) { each(f); });
  __syncthreads();
  if (tid < beam) {
    const bool real = s.out_i[tid] != 0x7fffffff;                // else a place nothing finite was left for: hypothesis 0, label 0
    score_out[q * beam + tid] = s.out_v[tid];
    src_out[q * beam + tid] = real ? s.out_i[tid] / V : 0;
    label_out[q * beam + tid] = real ? s.out_i[tid] % V : 0;
  }
}

// out[q * beam + k][0..width) = in[q * beam + src[q * beam + k]][0..width) for up to kGatherMax arrays in one launch.  Array i
// is copied in units of unit[i] bytes (16, 8, 4 or 2: the widest that its row length, leading dimensions and base addresses
// allow), one unit per thread; blocks [first_block[i], first_block[i+1]) work on array i.
constexpr int kGatherMax = 8;
struct GatherArgs {
  const char* in[kGatherMax]; char* out[kGatherMax];
  long ld_in[kGatherMax], ld_out[kGatherMax];          // bytes
  int units[kGatherMax], unit[kGatherMax];             // units per row; bytes per unit
  int first_block[kGatherMax + 1];
  int count, rows, beam;
  const int* src;
};
__global__ __launch_bounds__(256) void beam_gather_kernel(GatherArgs a) {
  int i = 0;
#pragma unroll
  for (int j = 1; j < kGatherMax; ++j)
    if (j < a.count && (int)blockIdx.x >= a.first_block[j]) i = j;
  const long idx = (long)((int)blockIdx.x - a.first_block[i]) * 256 + threadIdx.x;
  const int upr = a.units[i];
  if (idx >= (long)a.rows * upr) return;
  const int r = (int)(idx / upr), c = (int)(idx - (long)r * upr);
  int s = a.src[r];
  s = s < 0 ? 0 : (s >= a.beam ? a.beam - 1 : s);
  const int u = a.unit[i];
  const char* pi = a.in[i] + ((long)(r / a.beam) * a.beam + s) * a.ld_in[i] + (long)c * u;
  char* po = a.out[i] + (long)r * a.ld_out[i] + (long)c * u;
  if (u == 16) *(uint4*)po = *(const uint4*)pi;
  else if (u == 8) *(uint2*)po = *(const uint2*)pi;
  else if (u == 4) *(uint32_t*)po = *(const uint32_t*)pi;
  else *(uint16_t*)po = *(const uint16_t*)pi;
}

// trg[r] = W[label[r]] + b (bfloat16 table and result, float bias); labels outside [0, V) give the bias alone
__global__ void embed_kernel(const int* __restrict__ label, const uint16_t* __restrict__ W, const float* __restrict__ b,
                             uint16_t* __restrict__ out, long ld_out, int rows, int n, int V) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)rows * n) return;
  const int r = (int)(idx / n), c = (int)(idx % n);
  const int l = label[r];
  const float w = (l >= 0 && l < V) ? bf_bits2f(W[(long)l * n + c]) : 0.f;
  out[(long)r * ld_out + c] = f2bf_bits(w + (b ? b[c] : 0.f));
}

}  // namespace
}  // namespace lstm

using namespace lstm;

extern "C" {

static int beam_dims(int Q, int beam, int V) {
  if (Q < 0 || beam < 1 || V < 1 || (long)Q * beam > 0x7fffffffL / 16) return LSTM_ERR_DIM;
  if (beam > kBeamMax || V > kVocabMax) return LSTM_ERR_UNSUPPORTED;
  return LSTM_OK;
}

// Stretches a row is cut into: as many as the device holds at once (three work-groups a compute unit), of at least 2048 entries.
static int beam_parts(int Q, int beam, int V) {
  const long rows = (long)Q * beam;
  return rows < 1 ? 1 : (int)std::max(1L, std::min({(long)kRowParts, kRowGroups / rows, (long)V / 2048}));
}
static uint64_t beam_bytes(int Q, int beam, int parts) {
  const auto whole = [](uint64_t b) { return (b + 255) / 256 * 256; };
  const uint64_t rows = (uint64_t)Q * beam;
  return 256 + 2 * whole(rows * parts * beam * 4) + (parts > 1 ? whole(rows * parts * sizeof(float4)) : 0);
}

int lstm_beam_query(int Q, int beam, int V, uint64_t* workspace_bytes) {
  if (!workspace_bytes) return LSTM_ERR_NULL;
  const int rc = beam_dims(Q, beam, V);
  if (rc) return rc;
  *workspace_bytes = beam_bytes(Q, beam, beam_parts(Q, beam, V));
  return LSTM_OK;
}

// both kernels of a step; cand_val / cand_lab hold Q * beam * parts * beam entries each, part_sums Q * beam * parts
static int beam_launch(int Q, int beam, int V, const float* logits, int64_t ld, const float* score_in, float* score_out, int32_t* src,
                       int32_t* label, int parts, float* cand_val, int* cand_lab, float4* part_sums, hipStream_t st) {
  const int per = cdiv(cdiv(V, 4), parts), step = cdiv(per, cdiv(per, 256 * kRowPieces));       // pieces of a stretch, of a round
  const auto row = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(Q * beam * parts)), dim3(64 * waves), 0, st, logits, (long)ld, score_in, cand_val, cand_lab, part_sums, V,
                       beam, parts, per, step);
  };
  const int u = cdiv(step, 256);
  if (step <= 64) row(beam_row_kernel<1, 1>, 1);
  else if (u <= 1) row(beam_row_kernel<1, 4>, 4);
  else if (u <= 2) row(beam_row_kernel<2, 4>, 4);
  else if (u <= 4) row(beam_row_kernel<4, 4>, 4);
  else if (u <= 8) row(beam_row_kernel<8, 4>, 4);
  else if (u <= 12) row(beam_row_kernel<12, 4>, 4);
  else if (u <= 16) row(beam_row_kernel<16, 4>, 4);
  else if (u <= 20) row(beam_row_kernel<20, 4>, 4);
  else row(beam_row_kernel<kRowPieces, 4>, 4);
  const auto merge = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3(Q), dim3(64 * waves), 0, st, cand_val, cand_lab, part_sums, score_out, src, label, V, beam, parts);
  };
  const int c = beam * parts * beam;
  if (c <= 64) merge(beam_merge_kernel<1, 1>, 1);
  else if (c <= 256) merge(beam_merge_kernel<4, 1>, 1);
  else if (c <= 512) merge(beam_merge_kernel<2, 4>, 4);
  else if (c <= 1024) merge(beam_merge_kernel<4, 4>, 4);
  else merge(beam_merge_kernel<kRowParts * kBeamMax * kBeamMax / 256, 4>, 4);
  if (hipGetLastError() != hipSuccess) return LSTM_ERR_HIP;
  return LSTM_OK;
}

static int beam_step_args(int Q, int beam, int V, const float* logits, int64_t ld, const float* score_in, float* score_out, int32_t* src,
                          int32_t* label) {
  if (!logits || !score_in || !score_out || !src || !label) return LSTM_ERR_NULL;
  const int rc = beam_dims(Q, beam, V);
  if (rc) return rc;
  if (ld < V) return LSTM_ERR_DIM;
  if (((uintptr_t)logits | (uintptr_t)score_in | (uintptr_t)score_out | (uintptr_t)src | (uintptr_t)label) & 3) return LSTM_ERR_ALIGN;
  return LSTM_OK;
}

int lstm_beam_step(int Q, int beam, int V, const float* logits, int64_t ld, const float* score_in, float* score_out, int32_t* src,
                   int32_t* label, void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!workspace) return LSTM_ERR_NULL;
  int rc = beam_step_args(Q, beam, V, logits, ld, score_in, score_out, src, label);
  if (rc) return rc;
  if (workspace_bytes < beam_bytes(Q, beam, 1)) return LSTM_ERR_SIZE;
  int parts = beam_parts(Q, beam, V);
  if (workspace_bytes < beam_bytes(Q, beam, parts)) parts = 1;
  if (Q == 0) return LSTM_OK;
  if ((rc = device_ok())) return rc;
  char* ws = (char*)(((uintptr_t)workspace + 255) / 256 * 256);
  const size_t half = ((size_t)Q * beam * parts * beam * 4 + 255) / 256 * 256;
  return beam_launch(Q, beam, V, logits, ld, score_in, score_out, src, label, parts, (float*)ws, (int*)(ws + half), (float4*)(ws + 2 * half),
                     (hipStream_t)stream);
}

// The same step for callers that cannot allocate: the survivors of the rows (the only scratch of the step) go to a
// device array that is part of the library's image.  Its address on each device is looked up once, with that device
// current, and kept; host code never uses the array's name for anything else.
int lstm_beam_step_static(int Q, int beam, int V, const float* logits, int64_t ld, const float* score_in, float* score_out,
                          int32_t* src, int32_t* label, void* stream) {
  int rc = beam_step_args(Q, beam, V, logits, ld, score_in, score_out, src, label);
  if (rc) return rc;
  if ((uint64_t)Q * beam * beam > kStaticCands) return LSTM_ERR_SIZE;
  if (Q == 0) return LSTM_OK;
  if ((rc = device_ok())) return rc;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kStaticDevices) { (void)hipGetLastError(); return LSTM_ERR_HIP; }
  char* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
      void* p = nullptr;
      if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return LSTM_ERR_HIP; }
      g_static_ptr[dev] = p;
    }
    base = (char*)g_static_ptr[dev];
  }
  // every entry the merge reads is written by the row kernel of the same call: nothing has to be cleared
  static_assert(kRowGroups * (kBeamMax * 4 + sizeof(float4)) <= kStaticCands * 4, "rows in stretches: their sums behind their labels");
  return beam_launch(Q, beam, V, logits, ld, score_in, score_out, src, label, beam_parts(Q, beam, V), (float*)base, (int*)(base + kStaticCands * 4),
                     (float4*)(base + 2 * kStaticCands * 4 - kRowGroups * sizeof(float4)), (hipStream_t)stream);
}

int lstm_beam_gather_many(int Q, int beam, int count, const lstm_gather_item* items, const int32_t* src, void* stream) {
  if (!items || !src) return LSTM_ERR_NULL;
  if (count < 1 || count > kGatherMax) return LSTM_ERR_DIM;
  if (Q < 0 || beam < 1 || (long)Q * beam > 0x7fffffffL / 16) return LSTM_ERR_DIM;
  if ((uintptr_t)src & 3) return LSTM_ERR_ALIGN;
  GatherArgs a = {};
  a.count = count; a.rows = Q * beam; a.beam = beam; a.src = src;
  for (int i = 0; i < count; ++i) {
    const lstm_gather_item& it = items[i];
    if (!it.in || !it.out) return LSTM_ERR_NULL;
    if (it.width < 1 || it.ld_in < it.width || it.ld_out < it.width) return LSTM_ERR_DIM;
    if (it.elem_bytes != 2 && it.elem_bytes != 4) return LSTM_ERR_UNSUPPORTED;
    if (((uintptr_t)it.in | (uintptr_t)it.out) & (uintptr_t)(it.elem_bytes - 1)) return LSTM_ERR_ALIGN;
    if (it.in == it.out) return LSTM_ERR_UNSUPPORTED;             // rows are read while others are written
    const long row_bytes = (long)it.width * it.elem_bytes, lbi = (long)it.ld_in * it.elem_bytes, lbo = (long)it.ld_out * it.elem_bytes;
    const uintptr_t all = (uintptr_t)it.in | (uintptr_t)it.out | (uintptr_t)row_bytes | (uintptr_t)lbi | (uintptr_t)lbo;
    const int u = !(all & 15) ? 16 : !(all & 7) ? 8 : !(all & 3) ? 4 : 2;
    a.in[i] = (const char*)it.in; a.out[i] = (char*)it.out; a.ld_in[i] = lbi; a.ld_out[i] = lbo;
    a.unit[i] = u; a.units[i] = (int)(row_bytes / u);
    const long blocks = ((long)a.rows * a.units[i] + 255) / 256;
    if (blocks + a.first_block[i] > 0x7fffffffL) return LSTM_ERR_DIM;
    a.first_block[i + 1] = a.first_block[i] + (int)blocks;
  }
  if (Q == 0) return LSTM_OK;
  int rc = device_ok();
  if (rc) return rc;
  hipLaunchKernelGGL(beam_gather_kernel, dim3((unsigned)a.first_block[count]), dim3(256), 0, (hipStream_t)stream, a);
  if (hipGetLastError() != hipSuccess) return LSTM_ERR_HIP;
  return LSTM_OK;
}

int lstm_beam_gather(int elem_bytes, int Q, int beam, int width, const void* in, int64_t ld_in, const int32_t* src, void* out,
                     int64_t ld_out, void* stream) {
  if (!in || !src || !out) return LSTM_ERR_NULL;
  const lstm_gather_item it = {elem_bytes, width, in, ld_in, out, ld_out};
  return lstm_beam_gather_many(Q, beam, 1, &it, src, stream);
}

int lstm_embed(int B, int n, int V, const int32_t* label, const void* W_trg, const float* b_trg, void* out, int64_t ld_out, void* stream) {
  if (!label || !W_trg || !out) return LSTM_ERR_NULL;
  if (B < 0 || n < 1 || V < 1 || ld_out < n || (long)B * n > 0x7fffffffL) return LSTM_ERR_DIM;
  if ((((uintptr_t)W_trg | (uintptr_t)out) & 1) || (((uintptr_t)label | (uintptr_t)b_trg) & 3)) return LSTM_ERR_ALIGN;
  if (B == 0) return LSTM_OK;
  int rc = device_ok();
  if (rc) return rc;
  const long total = (long)B * n;
  hipLaunchKernelGGL(embed_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, label, (const uint16_t*)W_trg, b_trg,
                     (uint16_t*)out, (long)ld_out, B, n, V);
  if (hipGetLastError() != hipSuccess) return LSTM_ERR_HIP;
  return LSTM_OK;
}

}  // extern "C"
