// C entry points of the forward and backward micro-step: validate, then dispatch on dtype.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "loong_internal.h"

using namespace loong;

namespace {

// Step `t` of a run: valid by itself and equal to the first in all but the visiting chunk's ids.
int check_run(const loong_step_desc* descs, int t, StepGeom* g) {
  if (!descs) return fail(LOONG_E_NULL, "descriptor is NULL");
  if (int rc = check_step(&descs[t], g)) return rc;
  const loong_step_desc &a = descs[0], &b = descs[t];
  if (a.batch != b.batch || a.n_q_heads != b.n_q_heads || a.n_kv_heads != b.n_kv_heads || a.head_dim != b.head_dim ||
      a.q_len != b.q_len || a.kv_len != b.kv_len || a.chunk_len != b.chunk_len ||
      std::memcmp(a.q_chunk, b.q_chunk, sizeof(a.q_chunk)) || a.causal != b.causal || a.dtype != b.dtype ||
      a.softmax_scale != b.softmax_scale || a.flags != b.flags || std::memcmp(a.q_stride, b.q_stride, sizeof(a.q_stride)) ||
      std::memcmp(a.kv_stride, b.kv_stride, sizeof(a.kv_stride)) || std::memcmp(a.o_stride, b.o_stride, sizeof(a.o_stride)))
    return fail(LOONG_E_SHAPE, "step %d of a run differs from the first in more than its key chunks", t);
  return LOONG_OK;
}

// Steps of a valid run that go into one launch.  More steps hide more ramps and ragged ends, but the
// key-owning workgroups of a long launch drift apart and no longer find each other's query tiles in L2.  The run is
// cut into as many launches as its operations hold budgets of 9.4e9 head_dim (1.2e12 at 128, some 1.3 ms), and the steps
// are dealt out evenly, rounded up: no launch splits a step, and one may hold up to two budgets (two steps
// of 820 us below).  Backward passes with 1 / 2 / 4 / all steps per launch, and by the rule: 8 steps of 98 us (4 heads
// x 4096 rows) 788 / 693 / 546 / 469 us, 469; 8 of 420 us (8 x 8192 rows, one kv head) 3365 / 3336 / 3231 / 3341, 3342; 8 of 800
// us (4 x 16384) 6424 / 6436 / 6513 / 6779, 6437; 4 of 1010 us (8 x 16000 rows, head_dim 64) 4052 / 4510 / 4777 / 4817, 4058.
int steps_per_launch(const loong_step_desc& d, const StepGeom& g, double pairs, int n_steps) {
  const double flops = 14. * d.head_dim * pairs * d.n_q_heads * d.batch;
  const double per_launch = 9.4e9 * d.head_dim;
  const int launches = (int)std::max(std::min(std::ceil(flops / per_launch), (double)n_steps), std::ceil(n_steps / (double)kMaxSteps));
  const int per = (n_steps + launches - 1) / launches;
  return d.dtype == LOONG_FP32 ? per : (int)std::min<int64_t>(per, bwd_steps_that_fit_bf16(d, g));  // (every step has as many keys)
}

// A backward run, valid as a whole, cut into launches.
struct BwdRun {
  const loong_step_desc* descs;
  int n_steps, per_launch;
  StepGeom g[kMaxSteps];   // of the launch looked at last
  loong_step_desc d;       // the same: the first step's, and dq is written by the first launch alone

  int check(const loong_step_desc* descs_, int n_steps_) {
    descs = descs_; n_steps = n_steps_;
    double pairs = 0;
    StepGeom x;
    for (int t = 0; t < n_steps; ++t) {
      if (int rc = check_run(descs, t, &x)) return rc;
      for (int a = 0; a < x.nq; ++a) pairs += keys_of_rows(x, a) * x.q[a].len;
      if (t < kMaxSteps) g[t] = x;
    }
    d = descs[0];
    per_launch = steps_per_launch(d, x, pairs, n_steps);
    return LOONG_OK;
  }
  // The steps of the launch that starts at step t0 (right after check: of the first).
  int steps(int t0) const { return std::min(n_steps - t0, per_launch); }
  int look_at(int t0) {
    for (int t = 0; t < steps(t0); ++t)
      if (int rc = check_step(&descs[t0 + t], &g[t])) return rc;
    d = descs[0];
    if (t0 > 0) d.flags &= ~LOONG_OVERWRITE_DQ;
    return LOONG_OK;
  }
};

}  // namespace

extern "C" {

int loong_attn_step_fwd(const loong_step_desc* desc, const void* q, const void* k, const void* v,
                        float* out, float* lse, void* stream) {
  return loong_attn_steps_fwd(desc, 1, q, &k, &v, out, lse, nullptr, stream);
}

int loong_attn_steps_fwd(const loong_step_desc* descs, int32_t n_steps, const void* q, const void* const* k,
                         const void* const* v, float* out, float* lse, void* o, void* stream) {
  clear_error();
  if (n_steps < 1) return fail(LOONG_E_SHAPE, "loong_attn_steps_fwd: %d steps", n_steps);
  StepGeom g;
  for (int t = 0; t < n_steps; ++t)  // every step is validated before anything is enqueued
    if (int rc = check_run(descs, t, &g)) return rc;
  if (!q || !k || !v || !out || !lse) return fail(LOONG_E_NULL, "loong_attn_step_fwd: NULL tensor");
  bool aligned = aligned16(q) && aligned16(out) && aligned16(o);
  for (int t = 0; t < n_steps; ++t) {
    if (!k[t] || !v[t]) return fail(LOONG_E_NULL, "loong_attn_step_fwd: NULL tensor");
    aligned = aligned && aligned16(k[t]) && aligned16(v[t]);
  }
  if (!aligned) return fail(LOONG_E_ALIGN, "loong_attn_step_fwd: q/k/v/out must be 16-byte aligned");
  const loong_step_desc& d = *descs;
  const bool half = d.dtype != LOONG_FP32;
  const int64_t rows = (int64_t)d.batch * d.n_q_heads * d.q_len;
  if (o && !half && (d.o_stride[2] != d.head_dim || d.o_stride[1] != (int64_t)d.q_len * d.head_dim ||
                     (d.batch > 1 && d.o_stride[0] != d.n_q_heads * d.o_stride[1])))
    return fail(LOONG_E_UNSUPPORTED, "loong_attn_steps_fwd: the fp32 copy needs a contiguous out");
  if (rows == 0) return LOONG_OK;
  return half ? launch_fwd_bf16(descs, n_steps, q, k, v, out, lse, o, stream) : launch_fwd_f32(descs, n_steps, q, k, v, out, lse, o, stream);
}

int loong_attn_step_bwd(const loong_step_desc* desc, const void* q, const void* k, const void* v,
                        const void* o, const void* d_o, const float* lse, float* delta, float* dq,
                        float* dk, float* dv, void* workspace, int64_t workspace_bytes, void* stream) {
  return loong_attn_steps_bwd(desc, 1, q, &k, &v, o, d_o, lse, delta, dq, &dk, &dv, workspace, workspace_bytes, stream);
}

int loong_attn_steps_bwd(const loong_step_desc* descs, int32_t n_steps, const void* q, const void* const* k,
                         const void* const* v, const void* o, const void* d_o, const float* lse, float* delta,
                         float* dq, float* const* dk, float* const* dv, void* workspace, int64_t workspace_bytes,
                         void* stream) {
  clear_error();
  if (n_steps < 1) return fail(LOONG_E_SHAPE, "loong_attn_steps_bwd: %d steps", n_steps);
  BwdRun run;
  // every step is validated before anything is enqueued
  if (int rc = run.check(descs, n_steps)) return rc;
  const loong_step_desc* desc = descs;
  const bool only_dkv = desc->flags & LOONG_BWD_ONLY_DKV, only_dq = desc->flags & LOONG_BWD_ONLY_DQ;
  if (only_dkv && only_dq)
    return fail(LOONG_E_UNSUPPORTED, "loong_attn_step_bwd: LOONG_BWD_ONLY_DKV and LOONG_BWD_ONLY_DQ exclude each other");
  if (!q || !k || !v || !d_o || !lse || !delta || (!only_dkv && !dq) || (!only_dq && (!dk || !dv)))
    return fail(LOONG_E_NULL, "loong_attn_step_bwd: NULL tensor");
  for (int t = 0; t < n_steps; ++t)
    if (!k[t] || !v[t] || (!only_dq && (!dk[t] || !dv[t]))) return fail(LOONG_E_NULL, "loong_attn_step_bwd: NULL tensor");
  const bool want_delta = desc->flags & LOONG_COMPUTE_DELTA;
  if (want_delta && !o) return fail(LOONG_E_NULL, "loong_attn_step_bwd: LOONG_COMPUTE_DELTA needs o");
  bool aligned = aligned16(q) && aligned16(d_o) && (only_dkv || aligned16(dq)) && (!want_delta || aligned16(o));
  for (int t = 0; t < n_steps; ++t)
    aligned = aligned && aligned16(k[t]) && aligned16(v[t]) && (only_dq || (aligned16(dk[t]) && aligned16(dv[t])));
  if (!aligned) return fail(LOONG_E_ALIGN, "loong_attn_step_bwd: tensors must be 16-byte aligned");
  for (int t = 1; t < n_steps && !only_dq; ++t)  // the steps of a launch run in no order
    for (int u = 0; u < t; ++u)
      if (dk[t] == dk[u] || dv[t] == dv[u] || dk[t] == dv[u] || dv[t] == dk[u])
        return fail(LOONG_E_SHAPE, "loong_attn_steps_bwd: steps %d and %d have the same dk or dv", u, t);
  if (workspace_bytes < 0) return fail(LOONG_E_SHAPE, "loong_attn_step_bwd: negative workspace size");
  if (desc->batch == 0) return LOONG_OK;
  // (the counters are cleared once for all launches of the run that count: each leaves them zero)
  BwdPrologue before{want_delta ? o : nullptr, d_o, delta, nullptr};
  if (desc->dtype == LOONG_FP32) {
    if (int rc = launch_prologue(*desc, before, stream)) return rc;
    for (int t0 = 0; t0 < n_steps; t0 += run.per_launch) {
      if (int rc = t0 ? run.look_at(t0) : LOONG_OK) return rc;
      if (int rc = launch_bwd_f32(run.d, run.g, run.steps(t0), q, k + t0, v + t0, d_o, lse, delta, dq, only_dq ? nullptr : dk + t0,
                                  only_dq ? nullptr : dv + t0, stream))
        return rc;
    }
    return LOONG_OK;
  }
  // scratch for shared loops: checked before anything is enqueued.  (A run of one launch, as all short ones are, is looked at
  // and planned once: some 0.5 us for 4 steps, 2.5 for 32, which a call that asked for each size and planned again paid three times.)
  BwdPlan plan{};
  bool counts = false;
  for (int t0 = 0; t0 < n_steps; t0 += run.per_launch) {
    if (t0) {
      if (int rc = run.look_at(t0)) return rc;
      plan = {};
    }
    plan_bwd_bf16(run.d, run.g, run.steps(t0), &plan);
    if (const int64_t need = least_workspace_of(plan)) {
      if (!workspace)
        return fail(LOONG_E_NULL, "loong_attn_step_bwd: this step needs a workspace of %lld bytes (loong_workspace_bytes)",
                    (long long)need);
      if (!aligned16(workspace)) return fail(LOONG_E_ALIGN, "loong_attn_step_bwd: the workspace must be 16-byte aligned");
      if (workspace_bytes < need)
        return fail(LOONG_E_SHAPE, "loong_attn_step_bwd: workspace of %lld bytes, this step needs %lld (loong_workspace_bytes)",
                    (long long)workspace_bytes, (long long)need);
    }
    counts |= fit_bwd_bf16(&plan, workspace, workspace_bytes);
  }
  if (counts && !(desc->flags & LOONG_WORKSPACE_CLEAN)) before.head = workspace;
  for (int t0 = 0; t0 < n_steps; t0 += run.per_launch) {
    if (run.per_launch < n_steps) {
      if (int rc = run.look_at(t0)) return rc;
      plan = {};
      plan_bwd_bf16(run.d, run.g, run.steps(t0), &plan);
      fit_bwd_bf16(&plan, workspace, workspace_bytes);
    }
    if (int rc = launch_bwd_bf16(run.d, plan, run.steps(t0), t0 ? nullptr : &before, q, k + t0, v + t0, d_o, lse, delta, dq,
                                 only_dq ? nullptr : dk + t0, only_dq ? nullptr : dv + t0, workspace, stream))
      return rc;
  }
  return LOONG_OK;
}

int loong_workspace_bytes(const loong_step_desc* desc, int64_t* bytes) {
  return loong_workspace_bytes_steps(desc, 1, bytes);
}

int loong_workspace_bytes_steps(const loong_step_desc* descs, int32_t n_steps, int64_t* bytes) {
  clear_error();
  if (n_steps < 1) return fail(LOONG_E_SHAPE, "loong_workspace_bytes_steps: %d steps", n_steps);
  BwdRun run;
  if (int rc = run.check(descs, n_steps)) return rc;
  if (!bytes) return fail(LOONG_E_NULL, "loong_workspace_bytes: NULL result");
  *bytes = 0;
  if (descs->dtype == LOONG_FP32 || descs->batch == 0) return LOONG_OK;
  for (int t0 = 0; t0 < n_steps; t0 += run.per_launch) {
    if (int rc = t0 ? run.look_at(t0) : LOONG_OK) return rc;
    BwdPlan plan{};
    plan_bwd_bf16(run.d, run.g, run.steps(t0), &plan);
    *bytes = std::max(*bytes, workspace_of(plan));
  }
  return LOONG_OK;
}

}  // extern "C"
