// Exchange of partial results between the workgroups that share one tile's loop (several
// workgroups walk over parts of it; one adds the parts up).  Who adds is decided when the
// workgroups START: each claims a ticket, and the one that draws the last gathers.  All the others
// are running by then, so its wait for them ends whatever the order of dispatch; they park their
// parts in the caller's workspace, publish, and leave, while the gatherer keeps its own part in
// registers.  (Deciding at the end, by arrival, made every workgroup park its part and wait for the
// stores before it could count itself, and put the ticket's round trip after the loop instead
// of beside the first loads.)  The parts are added in split order, so the result does not depend on
// who gathers.
//
// The parts cross between XCDs, whose L2s are not coherent for ordinary accesses.  A device-scope
// fence would do (release: write back the XCD's L2, acquire: invalidate it), but every workgroup
// would pay for the whole cache (measured: 1.4-1.8x the time of a step).  Instead every word is
// stored and loaded with device scope (sc1), i.e. written through to and read from the level all
// XCDs share; the stores are waited for (vmcnt) before the workgroup publishes, and the gatherer's
// loads are issued after it has seen every part published.
//
// Counter of a tile: low half = tickets drawn, high half = parts published.  It must be zero
// before the launch and the gatherer leaves it zero.  If it is not (memory that two unordered calls share, or a
// caller that vouched for counters it never cleared), the tile's result is wrong, but nothing is read or written elsewhere and
// every wait ends; a wait that runs out stores NaN, so that most such mistakes show.
#pragma once
#include <hip/hip_runtime.h>

#include "device_utils.h"

namespace loong {

constexpr uint32_t kPublished = 0x10000u;

// One thread of the workgroup: draw a ticket; true for the gatherer of `n` workgroups (the last ticket; later ones are
// drawn from wrong counters only).
__device__ __forceinline__ bool claim_gather(uint32_t* cnt, int n) {
  const uint32_t before = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (before & (kPublished - 1)) >= (uint32_t)n - 1;
}

// One thread: this workgroup's part is in memory (every wave has waited for its stores, and a
// workgroup barrier has been passed since).
__device__ __forceinline__ void publish_part(uint32_t* cnt) {
  __hip_atomic_fetch_add(cnt, kPublished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One thread of the gatherer: wait for the other n - 1 parts and put the counter back to zero; false if they did not
// come.  The others started before this workgroup drew its ticket and have as many iterations of their loop left at most as it
// has done, so the wait is limited by that: 1024 looks per iteration and four million for everything else, which take 0.18 us
// each: 0.2 ms for an iteration of about 2 us, and 0.8 s.  (Looks are counted, not time: a wave that is taken off the device does not
// run out of them.)
constexpr int64_t kPolls = 1 << 22;
__device__ __forceinline__ bool await_parts(uint32_t* cnt, int n, int iterations) {
  bool all = false;
  for (int64_t left = kPolls + (int64_t)1024 * iterations; left > 0 && !all; --left) {
    all = (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16) == (uint32_t)n - 1;
    if (!all) __builtin_amdgcn_s_sleep(2);
  }
  __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return all;
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
