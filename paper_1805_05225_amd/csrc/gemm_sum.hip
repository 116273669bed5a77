// The second half of products whose K ranges stored their parts side by side: C (+)= bias + the sum of the parts, rows scattered, rounded once.
//
// A pass that reads every part once and takes 5 - 8 us, most of it a launch; so what a layer's backward pass has to add - the parts of dX, dW_x and
// dW_h and the slices of the bias gradient - is collected (SumList) and added in ONE launch (two layers of 330 units, 21 rows of at most 97
// frames, both directions: 4 launches and 26 us a layer fewer than a pass per product).
#include "common.h"

namespace lstm {
namespace {

// Four columns of a row per thread; parts in the order of their ranges.
__global__ __launch_bounds__(256) void add_parts_kernel(SumList l) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < SumList::kMax; ++i)
    if (i < l.count && (int)blockIdx.x >= l.first[i]) k = i;
  const SumJob g = l.j[k];
  const int b = (int)blockIdx.x - l.first[k], nq = (g.N + 3) / 4, per_z = (int)(((long)g.M * nq + 255) / 256), z = b / per_z;
  const long idx = (long)(b - z * per_z) * 256 + threadIdx.x;
  const int m = (int)(idx / nq), n = (int)(idx % nq) * 4;
  if (m >= (g.m_dev ? min(g.M, *g.m_dev) : g.M)) return;
  const float* p = g.parts + z * g.sPz + (long)m * g.ldp + n;                   // (ldp is a multiple of 4: whole quads)
  const long step = (long)g.M * g.ldp;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  int r = 0;
  for (; r + 8 <= g.ksplit; r += 8) {                                           // eight loads in flight
    f32x4 x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __builtin_nontemporal_load((const f32x4*)(p + (r + i) * step));
#pragma unroll
    for (int i = 0; i < 8; ++i) v += x[i];
  }
#pragma unroll 4
  for (; r < g.ksplit; ++r) v += __builtin_nontemporal_load((const f32x4*)(p + r * step));
  const float* bias = g.bias ? g.bias + g.sbiasz * z + n : nullptr;
  const long off = g.sCz * z + (long)(g.c_rows ? g.c_rows[m] : m) * g.ldc + n;
  const int cols = min(4, g.N - n);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < cols) v[i] += (bias ? bias[i] : 0.f) + (g.accumulate ? ((const float*)g.C)[off + i] : 0.f);
  if (g.out_bf16) {
    uint16_t* o = (uint16_t*)g.C + off;
    if (cols == 4 && ((uintptr_t)o & 7u) == 0) *(uint2*)o = make_uint2(f2bf_bits(v[0]) | ((unsigned)f2bf_bits(v[1]) << 16), f2bf_bits(v[2]) | ((unsigned)f2bf_bits(v[3]) << 16));
    else
      for (int i = 0; i < cols; ++i) o[i] = f2bf_bits(v[i]);
  } else {
    float* o = (float*)g.C + off;
    if (cols == 4 && ((uintptr_t)o & 15u) == 0) *(f32x4*)o = v;
    else
      for (int i = 0; i < cols; ++i) o[i] = v[i];
  }
}

}  // namespace

bool SumList::add(const SumJob& job) {
  if (count == kMax) return false;
  j[count] = job;
  first[count + 1] = first[count] + job.nz * (int)cdiv((long)job.M * ((job.N + 3) / 4), 256);
  ++count;
  return true;
}
hipError_t launch_sums(const SumList& l, hipStream_t s) {
  if (l.count == 0 || l.first[l.count] == 0) return hipSuccess;
  hipLaunchKernelGGL(add_parts_kernel, dim3(l.first[l.count]), dim3(256), 0, s, l);
  return hipGetLastError();
}
hipError_t finish_parts(const SumJob& job, size_t bytes, SumList* later, hipStream_t s) {
  if (later && later->add(job)) {
    later->used += (bytes + 255) / 256 * 256;
    return hipGetLastError();
  }
  SumList l;
  l.add(job);
  return launch_sums(l, s);
}

}  // namespace lstm
