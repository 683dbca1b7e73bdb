// Backward micro-step on the 16-bit matrix cores: launch planning and kernels.  The two halves of a
// step are the key-owning one (dK/dV of the visiting chunk, bwd_dkv_body.h) and the row-owning one
// (this step's share of dQ, bwd_dq_body.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "bwd_dkv_body.h"
#include "bwd_dq_body.h"
#include "device_utils.h"
#include "loong_internal.h"
#include "row_tiling.h"
#include "work_map.h"

namespace loong {
namespace {

__global__ __launch_bounds__(256) void zero_kernel(int64_t n4, float4* a, float4* b) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n4) {
    a[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    b[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// The arrival counters a launch with shared query loops uses start from zero: cleared on the
// caller's stream right before it (a fill kernel, so the call can be captured in a graph).
__global__ __launch_bounds__(256) void clear_counters_kernel(int n, uint32_t* cnt) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) cnt[i] = 0u;
}

// Work list of a step: key tiles per key segment (only segments some query can see), whether
// a key segment nobody sees exists (its gradients are cleared by the zero pass), and how many
// workgroups share the query loop of a key tile: more than one when the listed tiles are
// fewer than the compute units (`cus`), and twice as many when a diagonal block makes the loop
// lengths uneven.
struct SplitPlan {
  int nkt[2], kt_total, nsplit;
  bool unseen_keys;
  int64_t busy;  // listed key tiles x kv heads x batch
};

SplitPlan plan_split(const StepGeom& g, int G, int Hkv, int B, int q_len, int cus) {
  constexpr int BM = kBwdBM, BN = kBwdBN;
  SplitPlan s{};
  bool diag = false;
  for (int kb = 0; kb < 2; ++kb) {
    bool seen = false;
    if (kb < g.nk)
      for (int a = 0; a < g.nq; ++a) {
        seen |= g.cls[a][kb] != LOONG_SKIP && g.q[a].len > 0;
        diag |= g.cls[a][kb] == LOONG_DIAG;
      }
    s.nkt[kb] = seen ? (g.k[kb].len + BN - 1) / BN : 0;
    s.kt_total += s.nkt[kb];
    s.unseen_keys |= kb < g.nk && !seen && g.k[kb].len > 0;
  }
  s.busy = (int64_t)s.kt_total * Hkv * B;
  int nsplit = 1;
  const int64_t q_tiles = std::max<int64_t>((int64_t)G * ((q_len + BM - 1) / BM), 1);
  if (s.busy > 0 && s.busy < cus) nsplit = (int)std::min<int64_t>((cus + s.busy - 1) / s.busy, 16);
  if (diag && s.busy * nsplit <= 2 * cus) nsplit *= 2;
  // The last workgroup of a key tile adds up all its partial sums alone, at one CU's memory
  // rate (about 1.1 us per split), while a split shortens the loop by q_tiles x 1.9 us / n:
  // past n = sqrt(1.76 q_tiles) more splits lengthen the launch.
  nsplit = (int)std::min<int64_t>(nsplit, std::max<int64_t>(2, (int64_t)std::sqrt(1.76 * (double)q_tiles)));
  nsplit = (int)std::min<int64_t>(nsplit, q_tiles);
  if (s.busy > kWsCounters) nsplit = 1;  // (cannot happen: loops are only shared when key tiles are few)
  s.nsplit = nsplit;
  return s;
}

// bytes of partial sums one launch parks in the workspace
size_t partial_bytes(const SplitPlan& s, int head_dim) {
  return s.nsplit > 1 ? (size_t)s.busy * s.nsplit * kBwdWaves * (head_dim / 32) * 16 * 64 * sizeof(float) : 0;
}

// ---- kernels: the two halves of a step, alone and in one launch.  In the common launch the key-owning
// workgroups come first (they are the longer ones) and the row-owning ones fill the compute
// units as these finish: no gap and no second ramp between the halves, and where neither half has
// a workgroup for every unit they run side by side.  A whole step, two launches (and the passes that
// cleared counters and unseen keys) -> one: 2048 rows x 4096 keys x 8 heads 119.5 -> 116.2 us, the step
// of the same work whose keys are half unseen 135.3 -> 116.0, 3000 x 5000 without mask 315 -> 216,
// 400 rows x 200 keys x 4 heads 45 -> 19, 32768 x 16384 x 4 heads 3030 -> 3012.
template <class E, int D>
__global__ __launch_bounds__(kBwdWaves * 64) void bwd_dkv_kernel(const DkvParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BwdCfg<D>::SMEM_BYTES];
  dkv_body<E, D>(p, blockIdx.x, smem);
}

template <class E, int D, int KS>
__global__ __launch_bounds__(kRowWaves * 64) void dq_kernel(const DqParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DqCfg<D, KS>::SMEM_BYTES];
  dq_body<E, D, KS>(p, blockIdx.x, smem);
}

template <class E, int D, int KS>
__global__ __launch_bounds__(kBwdWaves * 64) void bwd_step_kernel(const DkvParams pk, const DqParams pq) {
  constexpr int BYTES = BwdCfg<D>::SMEM_BYTES > DqCfg<D, KS>::SMEM_BYTES ? BwdCfg<D>::SMEM_BYTES : DqCfg<D, KS>::SMEM_BYTES;
  static_assert(kBwdWaves == kRowWaves, "one workgroup size for both halves");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BYTES];
  if (blockIdx.x < pk.map.grid) dkv_body<E, D>(pk, blockIdx.x, smem);
  else dq_body<E, D, KS>(pq, blockIdx.x - pk.map.grid, smem);
}

// What a step enqueues: either half may be absent (flags, or nothing visible).
struct StepLaunch {
  DkvParams kv;
  DqParams q;
  bool do_kv, do_q;
};

// Key-owning half: work list, workspace and what is enqueued before it.
int plan_dkv(DkvParams& p, int flags, int D, void* workspace, int64_t workspace_bytes, hipStream_t st, bool* launch) {
  *launch = false;
  // Only key tiles that some query can see are listed (eight equal ranges of the list, one
  // per XCD, then carry equal work).
  const SplitPlan plan = plan_split(p.g, p.G, p.Hkv, p.B, p.q_len, planning_cus());
  p.nkt[0] = plan.nkt[0]; p.nkt[1] = plan.nkt[1]; p.kt_total = plan.kt_total;
  p.nsplit = plan.nsplit;
  p.accumulate = (flags & LOONG_ACCUM_DKV) ? 1 : 0;
  const int64_t total = plan.busy * plan.nsplit;
  if (total > 0x3ffffff0) return fail(LOONG_E_UNSUPPORTED, "backward grid too large");
  p.map = make_work_map((int64_t)p.Hkv * p.B, (int64_t)p.kt_total * plan.nsplit);
  if (plan.nsplit > 1) {  // (size and alignment were checked by the entry point, against the same plan)
    if (!workspace || workspace_bytes < kWsHeadBytes + (int64_t)partial_bytes(plan, D))
      return fail(LOONG_E_SHAPE, "loong_attn_step_bwd: workspace too small");
    p.ws_cnt = static_cast<uint32_t*>(workspace);
    p.ws_part = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + kWsHeadBytes);
  }
  if (total == 0) {
    if (plan.unseen_keys && !p.accumulate) {
      const int64_t n4 = (int64_t)p.B * p.Hkv * p.kv_len * D / 4;
      zero_kernel<<<dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st>>>(n4, reinterpret_cast<float4*>(p.dk),
                                                                            reinterpret_cast<float4*>(p.dv));
      return check_launch("loong_attn_step_bwd (clear dk/dv)");
    }
    return LOONG_OK;
  }
  if (plan.unseen_keys && !p.accumulate) {  // one of the two segments: the other one is listed
    const Segment& z = p.g.k[plan.nkt[0] == 0 ? 0 : 1];
    p.zero_start = z.start; p.zero_len = z.len;
  }
  if (plan.nsplit > 1 && !(flags & LOONG_WORKSPACE_CLEAN)) {
    clear_counters_kernel<<<dim3((unsigned)((plan.busy + 255) / 256)), dim3(256), 0, st>>>((int)plan.busy, p.ws_cnt);
    if (int rc = check_launch("loong_attn_step_bwd (clear counters)")) return rc;
  }
  *launch = true;
  return LOONG_OK;
}

template <class E, int D, int KS>
int launch_cfg(StepLaunch& s, hipStream_t st) {
  if (s.do_q) {
    DqParams& p = s.q;
    const RowTiling rt = make_row_tiling(p.g, p.G, p.Hq, p.B, kRowWaves / KS, /*list_blind=*/p.overwrite);
    p.GS = rt.GS; p.ntile[0] = rt.ntile[0]; p.ntile[1] = rt.ntile[1];
    p.tiles_total = rt.tiles_total; p.hgroups = rt.hgroups;
    if (rt.total_wg > 0x3ffffff0) return fail(LOONG_E_UNSUPPORTED, "backward (dQ) grid too large");
    p.map = make_work_map((int64_t)p.B * rt.hgroups, rt.tiles_total);
    s.do_q = rt.total_wg > 0;
  }
  const dim3 block(kBwdWaves * 64);
  if (s.do_kv && s.do_q && (int64_t)s.kv.map.grid + s.q.map.grid < 0x40000000)
    bwd_step_kernel<E, D, KS><<<dim3(s.kv.map.grid + s.q.map.grid), block, 0, st>>>(s.kv, s.q);
  else {
    if (s.do_kv) bwd_dkv_kernel<E, D><<<dim3(s.kv.map.grid), block, 0, st>>>(s.kv);
    if (s.do_q) dq_kernel<E, D, KS><<<dim3(s.q.map.grid), block, 0, st>>>(s.q);
  }
  return check_launch("loong_attn_step_bwd (bf16)");
}

template <class E>
int pick_cfg(StepLaunch& s, int head_dim, int ks, hipStream_t st) {
  if (head_dim == 128) {
    if (ks == 1) return launch_cfg<E, 128, 1>(s, st);
    if (ks == 2) return launch_cfg<E, 128, 2>(s, st);
    return launch_cfg<E, 128, 4>(s, st);
  }
  if (ks == 1) return launch_cfg<E, 64, 1>(s, st);
  if (ks == 2) return launch_cfg<E, 64, 2>(s, st);
  return launch_cfg<E, 64, 4>(s, st);
}

}  // namespace

int launch_bwd_bf16(const loong_step_desc& d, const StepGeom& g, const void* q, const void* k,
                    const void* v, const void* d_o, const float* lse, const float* delta, float* dq,
                    float* dk, float* dv, void* workspace, int64_t workspace_bytes, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  DeviceFacts dev;
  if (int rc = device_facts(&dev)) return rc;
  StepLaunch s{};
  s.do_kv = !(d.flags & LOONG_BWD_ONLY_DQ) && d.kv_len > 0;
  s.do_q = !(d.flags & LOONG_BWD_ONLY_DKV) && d.q_len > 0 && (d.kv_len > 0 || (d.flags & LOONG_OVERWRITE_DQ));
  if (s.do_kv) {
    DkvParams& p = s.kv;
    p.q = (const uint16_t*)q; p.k = (const uint16_t*)k; p.v = (const uint16_t*)v; p.d_o = (const uint16_t*)d_o;
    p.lse = lse; p.delta = delta; p.dk = dk; p.dv = dv;
    p.B = d.batch; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.G = d.n_q_heads / d.n_kv_heads;
    p.q_len = d.q_len; p.kv_len = d.kv_len;
    for (int i = 0; i < 3; ++i) { p.qs[i] = d.q_stride[i]; p.ks[i] = d.kv_stride[i]; }
    p.g = g; p.scale = d.softmax_scale; p.c = d.softmax_scale * kLog2e;
    if (int rc = plan_dkv(p, d.flags, d.head_dim, workspace, workspace_bytes, st, &s.do_kv)) return rc;
  }
  if (s.do_q) {
    DqParams& p = s.q;
    p.q = (const uint16_t*)q; p.k = (const uint16_t*)k; p.v = (const uint16_t*)v; p.d_o = (const uint16_t*)d_o;
    p.lse = lse; p.delta = delta; p.dq = dq;
    p.B = d.batch; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.G = d.n_q_heads / d.n_kv_heads;
    for (int i = 0; i < 3; ++i) { p.qs[i] = d.q_stride[i]; p.ks[i] = d.kv_stride[i]; p.os[i] = d.o_stride[i]; }
    p.q_len = d.q_len; p.g = g; p.scale = d.softmax_scale; p.c = d.softmax_scale * kLog2e;
    p.overwrite = (d.flags & LOONG_OVERWRITE_DQ) ? 1 : 0;
  }
  if (!s.do_kv && !s.do_q) return LOONG_OK;
  const int ks = pick_key_splits(g, d.n_q_heads / d.n_kv_heads, d.n_q_heads, d.batch, forced_key_splits(d.flags), dev.cus);
  if (d.dtype == LOONG_FP16) return pick_cfg<Fp16>(s, d.head_dim, ks, st);
  return pick_cfg<Bf16>(s, d.head_dim, ks, st);
}

int64_t bwd_workspace_bytes_bf16(const loong_step_desc& d, const StepGeom& g) {
  if (d.kv_len == 0 || d.batch == 0 || (d.flags & LOONG_BWD_ONLY_DQ)) return 0;
  const SplitPlan plan = plan_split(g, d.n_q_heads / d.n_kv_heads, d.n_kv_heads, d.batch, d.q_len, planning_cus());
  return plan.nsplit > 1 ? kWsHeadBytes + (int64_t)partial_bytes(plan, d.head_dim) : 0;
}

}  // namespace loong
