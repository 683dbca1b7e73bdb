// The visiting chunks a backward launch works on: one micro-step, or a run of micro-steps whose chunks
// are all resident.  The kernels take the table by value and index it with workgroup-uniform values
// (scalar loads, once per chunk).
#pragma once
#include <stdint.h>

namespace loong {

constexpr int kMaxSteps = 32;              // micro-steps per launch; longer runs take several launches
constexpr int kMaxHalves = 2 * kMaxSteps;  // key halves of their chunks

struct StepTable {
  const uint16_t *k[kMaxSteps], *v[kMaxSteps];
  float *dk[kMaxSteps], *dv[kMaxSteps];
  int klen;                        // keys per half; half 1 of a chunk starts at token klen
  // key halves, those some row sees first: step | half << 8 | class for q segment 0 << 10 | q segment 1 << 12
  uint32_t half[kMaxHalves];
  int n_seen, n_halves;
  // per q segment the halves it sees, in visit order: step | half << 8 | diagonal << 9
  uint32_t row_list[2][kMaxHalves];
  int n_list[2], n_diag[2];
};

constexpr uint32_t kDiagEntry = 1u << 9;

#ifdef __HIPCC__
__device__ __forceinline__ int entry_step(uint32_t e) { return (int)(e & 0xff); }
__device__ __forceinline__ int entry_half(uint32_t e) { return (int)(e >> 8) & 1; }
__device__ __forceinline__ int entry_class(uint32_t e, int qa) { return (int)(e >> (10 + 2 * qa)) & 3; }
#endif

}  // namespace loong
