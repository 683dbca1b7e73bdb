// Internal declarations shared by the host side of the library (not part of the ABI).
#pragma once
#include <stddef.h>
#include <stdint.h>
#include "loong.h"
#include "step_table.h"

namespace loong {

// Record an error text for the calling thread and hand back `code`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// A run of consecutive local tokens that belong to one global chunk.
struct Segment {
  int32_t start;   // first local token
  int32_t len;     // tokens
  int32_t chunk;   // global chunk id (only compared, never used as an address)
};

// Geometry of one micro-step after validation: up to two q segments and two key
// segments, and the class of every (q segment, key segment) block.
struct StepGeom {
  int32_t nq, nk;
  Segment q[2], k[2];
  uint8_t cls[2][2];
};

// Visible keys of the rows of q segment a, per row (half of a diagonal block)
inline double keys_of_rows(const StepGeom& g, int a) {
  double n = 0;
  for (int kb = 0; kb < g.nk; ++kb) n += g.cls[a][kb] == LOONG_FULL ? g.k[kb].len : g.cls[a][kb] == LOONG_DIAG ? 0.5 * g.k[kb].len : 0.;
  return n;
}

// Validate a descriptor (no device access).  Fills `g` when it succeeds.
int check_step(const loong_step_desc* d, StepGeom* g);

// 16-byte alignment test for device pointers.
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Map a hipError_t (as int) of the last launch to the ABI status.
int check_launch(const char* what);

// A launch takes fewer threads than this.  (The runtime refuses this very number; of larger ones it has run a part and
// reported success.)
constexpr int64_t kLaunchThreads = (int64_t)1 << 32;
inline bool launch_fits(int64_t workgroups, int threads) { return workgroups < kLaunchThreads / threads; }

// Facts of the current device, looked up once per device (device.hip).  device_facts fails with
// LOONG_E_HIP when there is no device and LOONG_E_UNSUPPORTED when it is not a gfx950 part.
struct DeviceFacts {
  int cus;  // compute units
};
int device_facts(DeviceFacts* f);
// Compute units to plan a launch for: the current device's, or those of an MI355X when no
// device can be asked (host-only size queries on a machine without a GPU).
constexpr int kDefaultCus = 256;
int planning_cus();

// Workspace of the backward step (caller-owned device memory): kWsCounters 32-bit arrival
// counters, then the partial sums.  A call that counts clears the counters on its own stream first (beside
// the delta it forms, else with a kernel of its own), so the memory may hold anything when it is handed in;
// with LOONG_WORKSPACE_CLEAN they are the caller's to have cleared.
constexpr int kWsCounters = 16384;
constexpr int64_t kWsHeadBytes = (int64_t)kWsCounters * 4;

// Key splits of the row-owning kernels forced through the descriptor's flags (0: automatic).
inline int forced_key_splits(int flags) {
  const int v = (flags >> LOONG_KEY_SPLITS_SHIFT) & 7;
  return v == 1 || v == 2 || v == 4 ? v : 0;
}

}  // namespace loong

// Kernel launchers (defined next to their kernels).  All arguments are already validated.
// The *_bf16 launchers serve both 16-bit storage types (LOONG_BF16 and LOONG_FP16).
namespace loong {
// (a valid run of `n` steps; `stored`: NULL, or where the result in the storage type goes too, contiguous; fp32: only if `out` is)
int launch_fwd_f32(const loong_step_desc* descs, int n, const void* q, const void* const* k, const void* const* v,
                   float* out, float* lse, void* stored, void* stream);
int launch_fwd_bf16(const loong_step_desc* descs, int n, const void* q, const void* const* k, const void* const* v,
                    float* out, float* lse, void* stored, void* stream);
// (`n` micro-steps that differ in the visiting chunk only, one geometry and one k, v, dk, dv each; n <= kMaxSteps)
int launch_bwd_f32(const loong_step_desc& d, const StepGeom* g, int n, const void* q, const void* const* k,
                   const void* const* v, const void* d_o, const float* lse, const float* delta, float* dq,
                   float* const* dk, float* const* dv, void* stream);
// What a backward call enqueues before its first launch: delta from `o`, unless that is NULL, and the counters at
// `head` cleared, unless that is NULL.
struct BwdPrologue {
  const void *o, *d_o;
  float* delta;
  void* head;
};
int launch_prologue(const loong_step_desc& d, const BwdPrologue& p, void* stream);
// How a launch over `n` micro-steps that differ in the visiting chunk only is divided (16-bit kernels).
struct BwdPlan {
  StepTable tab;             // (the chunks' pointers are the launch's)
  StepGeom rows;             // the q segments, and which of them see keys in any step
  int64_t busy;              // listed key tiles x kv heads x batch
  double per_cu, longest_row;  // multiply-adds per head_dim: all / CUs; of a row's keys
  int nkt;                   // tiles per key half
  int nsplit, nsplit_least;  // workgroups that share a key tile's query loop; with as little workspace as the launch can do with
  int ks, parts;             // row-owning half: key splits inside a workgroup; workgroups that share a tile's keys
  int64_t row_tiles;         // q tiles x head groups x batch
  int64_t key_bytes, least_bytes, row_bytes;  // partial sums of the key-owning half, at the least, and behind them of the row-owning half
};
inline int64_t workspace_of(const BwdPlan& p) { return p.key_bytes + p.row_bytes > 0 ? kWsHeadBytes + p.key_bytes + p.row_bytes : 0; }
inline int64_t least_workspace_of(const BwdPlan& p) {
  const int64_t b = p.key_bytes < p.least_bytes ? p.key_bytes : p.least_bytes;
  return b > 0 ? kWsHeadBytes + b : 0;
}
// (`plan`: zeroed)
void plan_bwd_bf16(const loong_step_desc& d, const StepGeom* g, int n, BwdPlan* plan);
// Gives up what a workspace of at least least_workspace_of() has no room for.  Does the launch count in it?
bool fit_bwd_bf16(BwdPlan* plan, const void* workspace, int64_t workspace_bytes);
// (a plan fitted to the workspace; `before`: enqueued first, once the launch is known to fit; or NULL)
int launch_bwd_bf16(const loong_step_desc& d, BwdPlan& plan, int n, const BwdPrologue* before, const void* q, const void* const* k,
                    const void* const* v, const void* d_o, const float* lse, const float* delta, float* dq,
                    float* const* dk, float* const* dv, void* workspace, void* stream);
// steps of a run that one launch has room for
int64_t bwd_steps_that_fit_bf16(const loong_step_desc& d, const StepGeom& g);
// delta of every row, and with `head` the counters of a workspace cleared; these alone
int launch_delta(const loong_step_desc& d, const void* o, const void* d_o, float* delta, void* head, void* stream);
int launch_clear_head(void* head, void* stream);
}  // namespace loong
