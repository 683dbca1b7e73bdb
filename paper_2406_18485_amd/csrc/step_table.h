// The visiting chunks a backward launch works on: one micro-step, or a run of micro-steps whose chunks
// are all resident.  The kernels take the table by value and index it with workgroup-uniform values
// (scalar loads, once per chunk).
//
// A look at a kernel argument is a round trip to memory, and one that needs the last one's answer pays again: entry,
// then step, then pointer made a key tile's prologue three looks longer.  So what a launch over one step reads (two
// entries, one step) lies at fixed places, is loaded together (scalar_now keeps the compiler from choosing an address
// first and loading then) and only later entries are looked up.  A whole step of 64 x 8 heads, 1 row x 1024 keys, head_dim 128:
// 321 -> 271 us, with the fragments of bwd_dkv_body.h requested together.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#endif

namespace loong {

constexpr int kMaxSteps = 32;              // micro-steps per launch; longer runs take several launches
constexpr int kMaxHalves = 2 * kMaxSteps;  // key halves of their chunks

struct StepTable {
  int klen;                        // keys per half; half 1 of a chunk starts at token klen
  int n_seen, n_halves;            // entries in `half`: those some row sees, all
  int n_list[2], n_diag[2];        // entries in `row` per q segment, and the diagonal ones among them
  uint32_t first_half[2], first_row[2][2];  // the first two of each list again, beside the counts
  struct Chunk {
    const uint16_t *k, *v;
    float *dk, *dv;
  } step[kMaxSteps];
  // key halves, those some row sees first: step | half << 8 | class for q segment 0 << 10 | q segment 1 << 12
  uint32_t half[kMaxHalves];
  // per q segment the halves it sees, in visit order: step | half << 8 | diagonal << 9
  uint32_t row[2][kMaxHalves];
};

constexpr uint32_t kDiagEntry = 1u << 9;

#ifdef __HIPCC__
__device__ __forceinline__ int entry_step(uint32_t e) { return (int)(e & 0xff); }
__device__ __forceinline__ int entry_half(uint32_t e) { return (int)(e >> 8) & 1; }
__device__ __forceinline__ int entry_class(uint32_t e, int qa) { return (int)(e >> (10 + 2 * qa)) & 3; }
__device__ __forceinline__ uint32_t scalar_now(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane(x); }
template <class T>
__device__ __forceinline__ T* scalar_now(T* p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return reinterpret_cast<T*>((uint64_t)scalar_now((uint32_t)(a >> 32)) << 32 | scalar_now((uint32_t)a));
}
#endif

}  // namespace loong
