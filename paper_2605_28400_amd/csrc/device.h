// Device helpers shared by the sweep kernels (sweep.hip, packed.hip).
#pragma once
#include "internal.h"

namespace trioseq {
namespace {

constexpr int kBufFlags = 0x00020000;       // raw buffer, gfx9 family
constexpr uint32_t kOob = 0xF0000000u;      // voffset outside every buffer

typedef __amdgpu_buffer_rsrc_t Rsrc;

__device__ __forceinline__ Rsrc make_rsrc(const void* p, uint64_t bytes) {
  const uint32_t n = bytes > 0x7FFFFFFFull ? 0x7FFFFFFFu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)n, kBufFlags);
}

__device__ __forceinline__ uint32_t residue_at(const uint32_t* __restrict__ words, uint64_t off,
                                               uint32_t p) {
  return (words[off + (p >> 4)] >> ((p & 15u) << 1)) & 3u;
}

__device__ __forceinline__ int sbyte(uint32_t tab, uint32_t sh) {
  return __builtin_amdgcn_sbfe((int)tab, sh, 8);
}

__device__ __forceinline__ int max3i(int a, int b, int c) { return max(max(a, b), c); }

__device__ __forceinline__ uint32_t pick4(uint32_t code, uint32_t t0, uint32_t t1, uint32_t t2,
                                          uint32_t t3) {
  return code == 0 ? t0 : code == 1 ? t1 : code == 2 ? t2 : t3;
}

constexpr int kTagAlways = 0x7FFFFFFF;

// A wait that gave up: the run's error flag is raised, and the release fence
// orders it before every store the wave issues afterwards. A panel that gave
// up goes on with whatever its faces hold, so the flag must become visible
// no later than the faces it writes from then on: a downstream panel that
// consumes them (and the panel that publishes the score after it) then sees
// the flag too.
__device__ __forceinline__ void raise_error(int* err) {
  if ((threadIdx.x & 63) == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
}

// The score of a split triplet, published by its last panel once the sweep is
// over: INT32_MIN if any wait of the run gave up. The acquire fence orders the
// flag's load after the face loads that the panel's result depends on.
__device__ __forceinline__ void publish_score(int32_t* so, int v, const int* err) {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const bool bad = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  // System scope: the score may live in mapped host memory (serving), where
  // the host picks it up while the kernel is still running.
  __hip_atomic_store(so, bad ? INT32_MIN : v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Start of a run, by one workgroup: next generation, error flag, queue head and
// finished counts cleared. A run takes `step` tags from its generation ctl[0]
// on; ctl[3] is the highest tag of the runs so far. Before the tags leave 31
// bits (after millions of runs) the pool of tagged faces is cleared, so that no
// old tag can look current, and they start over.
__device__ __forceinline__ void next_run(int* ctl, int* counter, int* pool, uint64_t pool_ints, int step) {
  const int last = ctl[3];
  const bool wrap = last >= kTagAlways - 2 * step;
  __syncthreads();
  if (wrap)
    for (uint64_t q = threadIdx.x; q < pool_ints; q += blockDim.x) pool[q] = 0;
  if (threadIdx.x == 0) {
    const int gen = (wrap ? 0 : last) + 1;
    ctl[0] = gen;
    ctl[1] = 0;
    ctl[3] = gen + step - 1;
    counter[0] = 0;
    counter[kFinished] = 0;
    counter[2 * kFinished] = 0;
  }
}

constexpr int kCohNone = 0;
constexpr int kCohDevice = 16;              // SC1

// A zero the compiler cannot see through. Re-reads of stale face entries add
// it to their scalar offset, so each retry is a distinct load that is neither
// merged with nor hoisted above an earlier one, while staying an ordinary
// (non-volatile) device-coherent load: all re-reads of a chunk are in flight
// together and share one wait.
__device__ __forceinline__ uint32_t opaque_zero() {
  uint32_t z;
  asm volatile("s_mov_b32 %0, 0" : "=s"(z));
  return z;
}

// Every wait for another wavefront is bounded (PanelIO::wait_ticks, 2 s by
// default, in ticks of the 100 MHz wall clock): past the limit the wave
// raises the error flag and proceeds (the score is then marked invalid), so a
// lost producer cannot hang the GPU.

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

// Four consecutive ints of LDS starting on a 16-byte boundary, read as one
// 128-bit access. A lane's halo row is either a ring row or a neighbour's
// slot row; both are 16-byte aligned, but the compiler cannot see that
// through the choice and would split the read into 8-byte halves, whose
// 16-byte lane stride makes lanes 8 apart collide on one LDS bank.
__device__ __forceinline__ v4i lds_v4(const int* p) {
  return *reinterpret_cast<const v4i*>(__builtin_assume_aligned(p, 16));
}

__device__ __forceinline__ int lds_get(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_put(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

}  // namespace
}  // namespace trioseq
