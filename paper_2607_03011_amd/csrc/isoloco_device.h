// Device helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "isoloco_kernels.h"

namespace isoloco {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum of one value per thread over a block of WAVES waves, in a fixed order
// (lds: WAVES doubles).  Result valid in thread 0.
template <int WAVES>
__device__ __forceinline__ double block_sum(double v, double* lds) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
    r = lds[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) r += lds[w];
  }
  return r;
}
__device__ __forceinline__ double block_sum256(double v, double* lds4) { return block_sum<4>(v, lds4); }

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}

// Word 3 of a raw buffer resource on CDNA3/CDNA4 (32-bit data format, no
// swizzle; the range check compares byte offsets with the record count).
constexpr int kBufferFlags = 0x00020000;
// Cache policy of the buffer loads of data read once (the "nt" bit).
constexpr int kStreamed = 2;

// A buffer resource over `bytes` bytes from p: loads at byte offsets at or
// past `bytes` return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kBufferFlags);
}

// Partials that one launch's workgroups hand to the last of them to arrive.
// They are stored and loaded with agent-scope atomics, which the hardware
// keeps coherent across the XCDs' separate L2 caches by themselves (no
// writeback or invalidation of a whole L2, which agent-scope release and
// acquire fences cost on this part).  arrive() waits for the workgroup's own
// store to complete before it counts itself, so that the workgroup that
// counts last finds every partial in place; it is called by one thread.
__device__ __forceinline__ void partial_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double partial_load(const double* p) {
  return __hip_atomic_load(const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Cache policy of buffer accesses at agent scope (the "sc1" bit): coherent
// across the XCDs like the atomics above.
constexpr int kAgentCoherent = 16;

// true in the workgroup that is the n-th to arrive at *cnt, which it sets back to zero
__device__ __forceinline__ bool arrive(int* cnt, int n) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const bool last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
  asm volatile("" ::: "memory");
  if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return last;
}

// The decisions of matrix mi from its Gram's norm partials (see NormMode,
// NormAction): the partials of its `nt` tiles are added in tile order.
__device__ __forceinline__ void norm_decide(const MatInfo& mi, const double* part, MatScalars& o, const NormArgs& a,
                                            int nt) {
  if (a.cls >= 0 && mi.sched != a.cls) return;
  const int act = a.mode == kNormFirst ? kActNone : a.action[mi.sched];
  if (a.mode != kNormFirst && act == kActNone) return;
  if (act == kActStop) {
    o.active = 0;
    return;
  }
  double s = 0.0;
  for (int x = 0; x < nt; ++x) s += partial_load(part + mi.norm_off + x);
  if (a.mode == kNormFirst) {
    o.gscale = ((o.flags & kFlagInput) == 0 && s > 0.0) ? (float)(1.0 / sqrt(sqrt(s))) : 0.f;
    return;
  }
  o.resid = (float)sqrt(s / mi.n);
  if (act == kActSwitch) {
    // stop at the end of this phase when every singular value is already at 1
    const bool go_on = (o.flags & kFlagInput) == 0 && !(o.resid <= a.tol_switch);
    // a matrix that still has a singular value away from 1 after the schedule
    // for a bound at the float32 resolution of Delta has one below it: its
    // direction in Q is decided by rounding, not by Delta
    if (go_on && a.flag_below[mi.sched]) o.flags |= kFlagBelowResolution;
    o.active = go_on ? 1 : 0;
    o.steps = go_on ? a.steps_total[mi.sched] : a.steps_here;
    o.qbuf = go_on ? a.buf_total[mi.sched] : a.buf_here;
  } else {
    if (a.flag_unconverged && !(o.resid <= 1e-3f) && (o.flags & kFlagInput) == 0) o.flags |= kFlagNotConverged;
    o.active = 0;
  }
}

}  // namespace isoloco
