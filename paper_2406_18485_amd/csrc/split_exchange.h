// Exchange of partial results between the workgroups that share one tile's loop (several
// workgroups walk over parts of it; one adds the parts up).  Every workgroup parks its part in the
// caller's workspace and then counts itself; the last to arrive adds the others' parts to its own,
// which it still has in registers (dQ: reads back), in split order, so the result does not depend on who that is.
// No workgroup waits for another: a launch ends whatever the counters hold.
//
// (Letting the last to START gather, chosen by a ticket drawn in the prologue, saves its parking but puts the
// ticket's round trip before the loop and needs a wait for the others' parts.  dK/dV alone, 4096 rows x 1024 keys, 8 heads on 2,
// head_dim 64: 45.9 us against 41.6 by arrival; 2 x 8 x 512 x 512: 18.3 against 15.3; whole backward steps 1-5 % longer.  Runs
// of steps go either way: 4 of 8 heads x 3998 rows 477 against 485, 4 of 16 heads x 606 rows 110 against 105.)
//
// The parts cross between XCDs, whose L2s are not coherent for ordinary accesses.  A device-scope
// fence would do (release: write back the XCD's L2, acquire: invalidate it), but every workgroup
// would pay for the whole cache (measured: 1.4-1.8x the time of a step).  Instead every word is
// stored and loaded with device scope (sc1), i.e. written through to and read from the level all
// XCDs share; the stores are waited for (vmcnt) before the workgroup counts itself, and the gatherer's
// loads are issued after its count has returned.
//
// The counter of a tile is zero before the launch and the last to arrive leaves it zero.  If it is not
// zero (memory that two unordered calls share, or a caller that vouched for counters it never cleared), the
// tile's result is wrong, but nothing is read or written elsewhere, and a count past the last gives NaN.
#pragma once
#include <hip/hip_runtime.h>

#include "device_utils.h"

namespace loong {

constexpr int kLeaves = 0, kGathers = 1, kCountsWrong = 2;

// One thread of the workgroup, whose part is in memory (every wave has waited for its stores, and a
// workgroup barrier has been passed since): what it does next.
__device__ __forceinline__ int arrive(uint32_t* cnt, int n) {
  const uint32_t before = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before < (uint32_t)n - 1) return kLeaves;
  __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return before == (uint32_t)n - 1 ? kGathers : kCountsWrong;
}

// 16 bytes per lane with device scope, as buffer accesses (the compiler counts them like any
// other): base uniform over the wave, byte offset per lane.
typedef uint32_t uintx4_t __attribute__((ext_vector_type(4)));
constexpr int kDeviceScope = 16;  // the sc1 bit of a buffer access
__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_buffer(void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00027000);
}
__device__ __forceinline__ void store_part(__amdgpu_buffer_rsrc_t buf, uint32_t off, floatx4_t x) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4_t, x), buf, off, 0, kDeviceScope);
}
__device__ __forceinline__ floatx4_t load_part(__amdgpu_buffer_rsrc_t buf, uint32_t off) {
  return __builtin_bit_cast(floatx4_t, __builtin_amdgcn_raw_buffer_load_b128(buf, off, 0, kDeviceScope));
}

}  // namespace loong
