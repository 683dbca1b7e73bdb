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

// workgroups that run on a compute unit together (registers, LDS) where a launch has enough of them
constexpr int wgs_per_unit(int head_dim) { return head_dim == 64 ? 2 : 1; }

constexpr double kLoopShare = 0.3;  // several steps per launch: a key tile's loop over the time of a unit
constexpr double kRowShare = 0.8;   // the same for the loop of a row-owning workgroup, which starts first

__global__ __launch_bounds__(256) void zero_kernel(int64_t n4, float4* a, float4* b) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n4) {
    a[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    b[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// bytes of partial sums one launch parks in the workspace
int64_t partial_bytes(int64_t busy, int nsplit, int head_dim) {
  return nsplit > 1 ? busy * nsplit * kBwdWaves * (head_dim / 32) * 16 * 64 * (int64_t)sizeof(float) : 0;
}

// Key-owning half, and work list of a launch over `n` micro-steps that differ in the visiting chunk only: the key halves some
// row sees and those nobody sees (their gradients are cleared), and how many workgroups share the query
// loop of a key tile.
void plan_split(const loong_step_desc& d, const StepGeom* g, int n, int cus, BwdPlan& s) {
  constexpr int BM = kBwdBM, BN = kBwdBN;
  const int G = d.n_q_heads / d.n_kv_heads, Hkv = d.n_kv_heads, B = d.batch, per_unit = wgs_per_unit(d.head_dim);
  StepTable* const tab = &s.tab;
  uint32_t entry[kMaxHalves];
  int64_t rows[kMaxHalves];
  int n_halves = 0, n_seen = 0, n_list[2] = {0, 0}, n_diag[2] = {0, 0};
  bool diag = false;
  double pairs = 0, most_keys = 0;
  int64_t most_rows = 0;
  for (int t = 0; t < n; ++t)
    for (int kb = 0; kb < g[t].nk; ++kb) {
      if (g[t].k[kb].len == 0) continue;
      uint32_t e = (uint32_t)t | (uint32_t)kb << 8;
      int64_t seen = 0;
      for (int a = 0; a < g[t].nq; ++a) {
        const int cls = g[t].cls[a][kb];
        e |= (uint32_t)cls << (10 + 2 * a);
        if (cls == LOONG_SKIP || g[t].q[a].len == 0) continue;
        seen += g[t].q[a].len;
        diag |= cls == LOONG_DIAG;
        tab->row[a][n_list[a]] = (uint32_t)t | (uint32_t)kb << 8 | (cls == LOONG_DIAG ? kDiagEntry : 0u);
        ++n_list[a];
        n_diag[a] += cls == LOONG_DIAG;
      }
      // halves with longer query loops first, visit order among equals, unseen ones last
      int at = n_halves++;
      for (; at > 0 && rows[at - 1] < seen && (n > 1 || rows[at - 1] == 0); --at) { rows[at] = rows[at - 1]; entry[at] = entry[at - 1]; }
      rows[at] = seen; entry[at] = e;
      n_seen += seen > 0;
      most_rows = std::max(most_rows, seen);
    }
  for (int a = 0; a < g[0].nq; ++a) {
    double keys = 0;
    for (int t = 0; t < n; ++t) keys += keys_of_rows(g[t], a);
    pairs += keys * g[0].q[a].len;
    most_keys = std::max(most_keys, keys);
  }
  const int klen = g[0].k[0].len;
  s.nkt = (klen + BN - 1) / BN;
  s.busy = (int64_t)n_seen * s.nkt * Hkv * B;
  // (the dK/dV half does 8 head_dim operations per pair, the dQ half 6)
  s.per_cu = 14. * pairs * G * Hkv * B / cus;
  s.longest_row = 6. * most_keys;
  tab->klen = klen; tab->n_seen = n_seen; tab->n_halves = n_halves;
  for (int i = 0; i < n_halves; ++i) tab->half[i] = entry[i];
  for (int a = 0; a < 2; ++a) { tab->n_list[a] = n_list[a]; tab->n_diag[a] = n_diag[a]; }
  for (int i = 0; i < 2; ++i) {
    tab->first_half[i] = tab->half[i];
    for (int a = 0; a < 2; ++a) tab->first_row[a][i] = tab->row[a][i];
  }
  const int64_t q_tiles = std::max<int64_t>((int64_t)G * ((d.q_len + BM - 1) / BM), 1);
  // The last workgroup of a key tile adds up all its partial sums alone, at one CU's memory
  // rate (about 1.1 us per split), while a split shortens the loop by q_tiles x 1.9 us / n:
  // past n = sqrt(1.76 q_tiles) more splits lengthen the launch.
  auto at_most = [&](int nsplit) {
    nsplit = (int)std::min<int64_t>(nsplit, std::max<int64_t>(2, (int64_t)std::sqrt(1.76 * (double)q_tiles)));
    nsplit = (int)std::min<int64_t>(nsplit, q_tiles);
    return s.busy > kWsCounters ? 1 : nsplit;  // (cannot happen for one step: loops are only shared when key tiles are few)
  };
  s.nsplit = s.nsplit_least = 1;
  if (n == 1) {
    // one step: more than one workgroup when the listed tiles are fewer than the compute units, and
    // twice as many when a diagonal block makes the loop lengths uneven
    int nsplit = 1;
    if (s.busy > 0 && s.busy < cus) nsplit = (int)std::min<int64_t>((cus + s.busy - 1) / s.busy, 16);
    auto uneven = [&](int nsplit) { return diag && s.busy * nsplit <= 2 * cus ? 2 * nsplit : nsplit; };  // (at head_dim 64 at most 1024 parts of 64 KB: the static scratch holds them)
    s.nsplit_least = at_most(uneven(nsplit));
    // Where the chip holds more workgroups than units (head_dim 64), loops that stay long are split until it is full; the exchange
    // costs some 12 us.  dK/dV alone, a workgroup per unit / a full chip: 128 tiles in a loop, 8 heads on 2 x 2000 rows x 20000 keys
    // 247 / 219 us; 256 tiles in either of two, 8192 x 8192 310 / 276; 32 and 24 tiles 67 / 69 and 53 / 53; 8 tiles (8 heads on 2 x
    // 121 x 20787) 23 / 35.  (With a workspace that has no room for it a workgroup per unit will do.)
    if (s.busy > 0 && s.busy * nsplit < (int64_t)per_unit * cus && q_tiles / nsplit >= 48)
      nsplit = (int)std::min<int64_t>((per_unit * cus + s.busy - 1) / s.busy, 16);
    s.nsplit = at_most(uneven(nsplit));
  } else if (s.busy > 0) {
    // Several steps: the tiles fill the chip; as many parts as make the longest loop a small part of a unit's time, or fewer
    // where these would end clearly earlier.  An estimate of that: all work dealt out over the places the chip has for workgroups, and then the
    // longest single workgroup, started as the last place falls free; in tiles of a query loop (some 1.9 us).  A workgroup's
    // prologue and stores are worth 3; parking and adding up shared sums 4 more and half a tile per part when the whole chip
    // does it, one more for a single workgroup.  A backward pass, without the estimate -> with it: 8 steps of 2 heads x 2000 rows 131 -> 104
    // us, 16 of 4 x 1000 137 -> 100, 3 of 12 x 1400 (head_dim 64) 61 -> 57, 8 of 8 x 1200 137 -> 120, 4 of 32 x 600 113 -> 88, 32 of 2 x
    // 638 x batch 2 188 -> 87.  Of 670 runs of 2 to 32 steps of 96 to 11000 rows, each timed with every number of parts, it takes 1.5 to
    // 2 % longer than the best on average (6 to 9 % without it), and sixteen of them 2-9 % longer than without it: how the parts and the
    // workgroups of the dQ half, which come first, fill the last places is not in it (6 steps of 3 heads on 1 x 1268 rows: four parts 56 us, the
    // six it takes 69).  (With a quarter of
    // the longest workgroup instead of all of it 2.5 % and up to 14 % longer than without, as 3 steps of 6 heads on 2 x 4430 rows x batch 2
    // 643 -> 671.  The estimate alone makes five parts of four on 8 steps of 4 x 16384 rows: 3.6 % longer.)
    const int most = (int)std::min(std::max(std::ceil(8. * BN * most_rows * G / (kLoopShare * s.per_cu)), 1.), 16.);
    const double loops = pairs * G * Hkv * B / ((double)BN * BM), longest = ((double)most_rows / BM + 1.) * G;  // tiles of all loops, of the longest (with its ragged ends)
    auto time = [&](int k) {
      return (loops + s.busy * k * (k == 1 ? 3. : 7. + 0.5 * k)) / (per_unit * cus) + longest / k + (k == 1 ? 3. : 4.);
    };
    int nsplit = most;
    double best = 0.97 * time(most);
    for (int k = 1; k < most; ++k)
      if (time(k) <= best) { best = time(k); nsplit = k; }
    s.nsplit = at_most(nsplit);
    s.nsplit_least = 1;  // (the estimate is about speed: with less room than it asks for, fewer parts will do)
  }
}

// The q segments of a launch, and which of them see keys in any of its steps (which is what the row tiling asks).
StepGeom seen_rows(const StepGeom* g, int n) {
  StepGeom rows = g[0];
  for (int t = 1; t < n; ++t)
    for (int a = 0; a < g[t].nq; ++a)
      if (segment_sees_keys(g[t], a)) rows.cls[a][0] = LOONG_FULL;
  return rows;
}

// Few rows and many keys: the loop over the keys of a q tile is the longest thing in the launch and most units have nothing to do,
// so several workgroups share it.  A part keeps at least 12 tiles: parking and adding up take some 10 us, as long as 8 tiles (24 instead of 12: 115 us for the first run).
// Whole backward steps, one workgroup -> several per tile: 121 rows x 20787 keys, 8 heads on 2, 232 -> 75 us (head_dim 64: 144 -> 44), 2 x 2
// heads x 300 x 8000 101 -> 54; runs of 32 steps, 2 heads x 200 rows 115 -> 55, 1 x 600 142 -> 54; 8 x 60 x 3000 26.7 -> 26.9.
// Only where both halves run: the dQ half alone needs no workspace.
void plan_rows(const loong_step_desc& d, int n, bool do_kv, int cus, BwdPlan& r) {
  const int G = d.n_q_heads / d.n_kv_heads;
  r.ks = forced_key_splits(d.flags);
  if (!r.ks && n > 1 && do_kv) {
    // several steps: the tallest row tiles whose loop still fits beside the other work of a unit
    for (r.ks = 1; r.ks < 4 && r.longest_row * (32 * kRowWaves / r.ks) > kRowShare * r.per_cu;) r.ks *= 2;
  }
  if (!r.ks) r.ks = pick_key_splits(r.rows, G, d.n_q_heads, d.batch, 0, cus * (do_kv ? wgs_per_unit(d.head_dim) : 1));
  r.row_tiles = make_row_tiling(r.rows, G, d.n_q_heads, d.batch, kRowWaves / r.ks, /*list_blind=*/d.flags & LOONG_OVERWRITE_DQ).total_wg;
  r.parts = 1;
  if (do_kv && r.row_tiles > 0 && 2 * r.row_tiles <= cus) {
    const double loop = r.longest_row / 6. / (r.ks == 1 ? 64 : 32 * r.ks);  // tiles of keys
    r.parts = (int)std::max<int64_t>(std::min<int64_t>({cus / r.row_tiles, (int64_t)(loop / 12.), 16}), 1);
    if (r.parts > 1) r.row_bytes = r.row_tiles * r.parts * (kRowWaves / r.ks) * 32 * d.head_dim * (int64_t)sizeof(float);
    // (a step that fits the static scratch goes on fitting; runs do not go there)
    if (r.busy + r.row_tiles > kWsCounters || (n == 1 && kWsHeadBytes + r.key_bytes + r.row_bytes > LOONG_STATIC_SCRATCH_BYTES)) {
      r.parts = 1;
      r.row_bytes = 0;
    }
  }
}

// ---- kernels: the two halves of a step, alone and in one launch.  In the common launch of one step the
// key-owning workgroups come first (they are the longer ones) and the row-owning ones fill the compute
// units as these finish: no gap and no second ramp between the halves, and where neither half has
// a workgroup for every unit they run side by side.  A whole step, two launches (and the passes that
// cleared counters and unseen keys) -> one: 2048 rows x 4096 keys x 8 heads 125.1 -> 118.3 us, the step
// of the same work whose keys are half unseen 136.6 -> 124.5, 3000 x 5000 without mask 317 -> 211,
// 400 rows x 200 keys x 4 heads 33 -> 20, 32768 x 16384 x 4 heads 3123 -> 3084.
// With several steps in the launch the row-owning workgroups are the longer ones (their loop runs over the
// keys of every step, dQ stays in registers throughout) and come first; the key tiles of all
// steps fill the chip, so few query loops are shared and one ramp and one ragged end serve all steps.
// A backward pass, a launch per step -> the run: 8 steps of 2048 rows x 4096 keys x 8 heads 1003 -> 851 us, 32 steps of
// 2048 rows x 4 heads, one kv head 1395 -> 529, 4 steps of 400 rows x 4 heads 158 -> 77 (with its forward).
// (Key-owning workgroups first in a run: 7 % slower at 8 x 2048 rows.)
template <class E, int D, int W>
__global__ __launch_bounds__(kBwdWaves * 64, 2 * W) void bwd_dkv_kernel(const StepTable tab, const DkvParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BwdCfg<D, W>::SMEM_BYTES];
  dkv_body<E, D, W>(tab, p, blockIdx.x, smem);
}

template <class E, int D, int KS, int W>
__global__ __launch_bounds__(kRowWaves * 64, 2 * W) void dq_kernel(const StepTable tab, const DqParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DqCfg<D, KS, W>::SMEM_BYTES];
  dq_body<E, D, KS, W>(tab, p, blockIdx.x, smem);
}

template <class E, int D, int KS, int W>
__global__ __launch_bounds__(kBwdWaves * 64, 2 * W) void bwd_step_kernel(const StepTable tab, const DkvParams pk, const DqParams pq) {
  constexpr int BYTES = BwdCfg<D, W>::SMEM_BYTES > DqCfg<D, KS, W>::SMEM_BYTES ? BwdCfg<D, W>::SMEM_BYTES : DqCfg<D, KS, W>::SMEM_BYTES;
  static_assert(kBwdWaves == kRowWaves, "one workgroup size for both halves");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[BYTES];
  const bool second = blockIdx.x >= pq.first_grid;
  const uint32_t block = blockIdx.x - (second ? pq.first_grid : 0u);
  if (second == pq.rows_first) dkv_body<E, D, W>(tab, pk, block, smem);
  else dq_body<E, D, KS, W>(tab, pq, block, smem);
}

// What a launch enqueues: either half may be absent (flags, or nothing visible).
struct StepLaunch {
  DkvParams kv;
  DqParams q;
  bool do_kv, do_q;
  bool clear;      // nobody sees any key: dk and dv of all steps are cleared
};

// Workgroups that a launch has room for.
constexpr int64_t kMaxGrid = kLaunchThreads / (kBwdWaves * 64) - 1;

// Key-owning half: work list and workspace.
int plan_dkv(StepLaunch& s, const BwdPlan& plan, int flags, void* workspace) {
  DkvParams& p = s.kv;
  s.do_kv = false;
  // Only key tiles that some query can see are listed (eight equal ranges of the list, one
  // per XCD, then carry equal work).
  p.nkt = plan.nkt; p.kt_total = plan.tab.n_seen * plan.nkt;
  p.nsplit = plan.nsplit;
  p.accumulate = (flags & LOONG_ACCUM_DKV) ? 1 : 0;
  const int64_t total = plan.busy * plan.nsplit;
  if (total > kMaxGrid) return fail(LOONG_E_UNSUPPORTED, "backward grid too large");
  if (total == 0) {
    s.clear = !p.accumulate;
    return LOONG_OK;
  }
  p.map = make_work_map((int64_t)p.Hkv * p.B, (int64_t)p.kt_total * plan.nsplit);
  if (p.map.grid > kMaxGrid) return fail(LOONG_E_UNSUPPORTED, "backward grid too large");
  if (plan.nsplit > 1) {  // (the entry point has fitted the plan to the workspace)
    p.ws_cnt = static_cast<uint32_t*>(workspace);
    p.ws_part = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + kWsHeadBytes);
  }
  s.do_kv = true;
  return LOONG_OK;
}

// Row-owning half: work list and workspace.
int plan_dq(StepLaunch& s, const BwdPlan& plan, void* workspace) {
  DqParams& p = s.q;
  const RowTiling rt = make_row_tiling(plan.rows, p.G, p.Hq, p.B, kRowWaves / plan.ks, /*list_blind=*/p.overwrite);
  p.parts = plan.parts;
  if (p.parts > 1) {
    p.ws_cnt = static_cast<uint32_t*>(workspace) + (kWsCounters - plan.row_tiles);  // (the other half counts from the front)
    p.ws_part = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + kWsHeadBytes + plan.key_bytes);
  }
  p.GS = rt.GS; p.ntile[0] = rt.ntile[0]; p.ntile[1] = rt.ntile[1];
  p.tiles_total = rt.tiles_total; p.hgroups = rt.hgroups;
  s.do_q = rt.total_wg > 0;
  if (!s.do_q) return LOONG_OK;
  if (rt.total_wg * p.parts > kMaxGrid) return fail(LOONG_E_UNSUPPORTED, "backward (dQ) grid too large");
  p.map = make_work_map((int64_t)p.B * rt.hgroups, (int64_t)rt.tiles_total * p.parts);
  if (p.map.grid > kMaxGrid) return fail(LOONG_E_UNSUPPORTED, "backward (dQ) grid too large");
  return LOONG_OK;
}

template <class E, int D, int KS, int W>
int launch_cfg(StepLaunch& s, const StepTable& tab, hipStream_t st) {
  const dim3 block(kBwdWaves * 64);
  if (s.do_kv && s.do_q && (int64_t)s.kv.map.grid + s.q.map.grid <= kMaxGrid) {
    s.q.first_grid = s.q.rows_first ? s.q.map.grid : s.kv.map.grid;
    bwd_step_kernel<E, D, KS, W><<<dim3(s.kv.map.grid + s.q.map.grid), block, 0, st>>>(tab, s.kv, s.q);
  } else {
    if (s.do_kv) bwd_dkv_kernel<E, D, W><<<dim3(s.kv.map.grid), block, 0, st>>>(tab, s.kv);
    if (s.do_q) dq_kernel<E, D, KS, W><<<dim3(s.q.map.grid), block, 0, st>>>(tab, s.q);
  }
  return check_launch("loong_attn_step_bwd (bf16)");
}

// head_dim 64 has two forms of either half, with the same results: for two workgroups per unit, and one with the registers, the
// look-ahead and the LDS of a unit to itself for launches that put hardly more than one on any.  Whole steps, one / two: 190 x 190 x 8
// heads 12.0 / 12.4 us, 512 x 512 x 8 14.4 / 14.8, 1554 rows of a diagonal step, 4 heads on 1 (280 workgroups) 28.3 / 31.0; 700 x 2000 x
// 4 (300) 30.9 / 27.7, 1024 x 1024, 16 heads on 4 37.6 / 31.8.  dQ alone: 2048 x 16384, 4 heads on 1 95 / 105, 700 x 900 x 4 x 16
// heads on 2 (352) 34.3 / 28.5; with a diagonal block, whose loops are uneven, 512 workgroups 209 / 245.  dK/dV alone: 1500 x 1500, 6 heads on 2 (264) 37.5 / 35.5.
template <class E, int D, int KS>
int launch_form(StepLaunch& s, const StepTable& tab, int cus, hipStream_t st) {
  if constexpr (D == 64) {
    const int64_t total = (int64_t)(s.do_kv ? s.kv.map.grid : 0) + (s.do_q ? s.q.map.grid : 0);
    const bool uneven = !s.do_kv && tab.n_diag[0] + tab.n_diag[1] > 0;
    if (total > (s.do_kv && s.do_q ? cus * 9 / 8 : cus) && !uneven) return launch_cfg<E, D, KS, 2>(s, tab, st);
  }
  return launch_cfg<E, D, KS, 1>(s, tab, st);
}

template <class E>
int pick_cfg(StepLaunch& s, const StepTable& tab, int head_dim, int ks, int cus, hipStream_t st) {
  if (head_dim == 128) {
    if (ks == 1) return launch_form<E, 128, 1>(s, tab, cus, st);
    if (ks == 2) return launch_form<E, 128, 2>(s, tab, cus, st);
    return launch_form<E, 128, 4>(s, tab, cus, st);
  }
  if (ks == 1) return launch_form<E, 64, 1>(s, tab, cus, st);
  if (ks == 2) return launch_form<E, 64, 2>(s, tab, cus, st);
  return launch_form<E, 64, 4>(s, tab, cus, st);
}

}  // namespace

void plan_bwd_bf16(const loong_step_desc& d, const StepGeom* g, int n, BwdPlan* plan) {
  const int cus = planning_cus();
  plan_split(d, g, n, cus, *plan);
  const bool do_kv = !(d.flags & LOONG_BWD_ONLY_DQ) && plan->busy > 0;
  plan->key_bytes = do_kv ? partial_bytes(plan->busy, plan->nsplit, d.head_dim) : 0;
  plan->least_bytes = do_kv ? partial_bytes(plan->busy, plan->nsplit_least, d.head_dim) : 0;
  plan->rows = seen_rows(g, n);
  plan->row_bytes = 0;
  if (!(d.flags & LOONG_BWD_ONLY_DKV) && d.q_len > 0) plan_rows(d, n, do_kv, cus, *plan);
}

bool fit_bwd_bf16(BwdPlan* p, const void* workspace, int64_t workspace_bytes) {
  const int64_t room = workspace && aligned16(workspace) ? workspace_bytes - kWsHeadBytes : 0;
  if (p->key_bytes > std::max<int64_t>(room, 0)) {  // as many parts as there is room for
    const int64_t part = p->key_bytes / p->nsplit;
    p->nsplit = std::max(p->nsplit_least, (int)(std::max<int64_t>(room, 0) / part));
    p->key_bytes = p->nsplit > 1 ? part * p->nsplit : 0;
  }
  if (p->row_bytes > 0 && p->key_bytes + p->row_bytes > room) {
    p->parts = 1;
    p->row_bytes = 0;
  }
  return p->key_bytes + p->row_bytes > 0;
}

int launch_bwd_bf16(const loong_step_desc& d, BwdPlan& plan, int n, const BwdPrologue* before, const void* q, const void* const* k,
                    const void* const* v, const void* d_o, const float* lse, const float* delta, float* dq,
                    float* const* dk, float* const* dv, void* workspace, void* stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  DeviceFacts dev;
  if (int rc = device_facts(&dev)) return rc;
  const int G = d.n_q_heads / d.n_kv_heads;
  StepLaunch s{};
  s.do_kv = !(d.flags & LOONG_BWD_ONLY_DQ) && d.kv_len > 0;
  s.do_q = !(d.flags & LOONG_BWD_ONLY_DKV) && d.q_len > 0 && (d.kv_len > 0 || (d.flags & LOONG_OVERWRITE_DQ));
  for (int t = 0; t < n; ++t) {
    StepTable::Chunk& c = plan.tab.step[t];
    c.k = (const uint16_t*)k[t]; c.v = (const uint16_t*)v[t];
    if (s.do_kv) { c.dk = dk[t]; c.dv = dv[t]; }
  }
  if (s.do_kv) {
    DkvParams& p = s.kv;
    p.q = (const uint16_t*)q; p.d_o = (const uint16_t*)d_o;
    p.lse = lse; p.delta = delta;
    p.B = d.batch; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.G = G;
    p.q_len = d.q_len; p.kv_len = d.kv_len;
    for (int i = 0; i < 3; ++i) { p.qs[i] = d.q_stride[i]; p.ks[i] = d.kv_stride[i]; }
    p.nq = plan.rows.nq; p.qseg[0] = plan.rows.q[0]; p.qseg[1] = plan.rows.q[1];
    p.scale = d.softmax_scale; p.c = d.softmax_scale * kLog2e;
    if (int rc = plan_dkv(s, plan, d.flags, workspace)) return rc;
  }
  if (s.do_q) {
    DqParams& p = s.q;
    p.q = (const uint16_t*)q; p.d_o = (const uint16_t*)d_o;
    p.lse = lse; p.delta = delta; p.dq = dq;
    p.B = d.batch; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.G = G;
    for (int i = 0; i < 3; ++i) { p.qs[i] = d.q_stride[i]; p.ks[i] = d.kv_stride[i]; p.os[i] = d.o_stride[i]; }
    p.q_len = d.q_len; p.qseg[0] = plan.rows.q[0]; p.qseg[1] = plan.rows.q[1];
    p.scale = d.softmax_scale; p.c = d.softmax_scale * kLog2e;
    p.overwrite = (d.flags & LOONG_OVERWRITE_DQ) ? 1 : 0;
    p.rows_first = n > 1;
  }
  if (s.do_q)
    if (int rc = plan_dq(s, plan, workspace)) return rc;
  const int64_t n4 = (int64_t)d.batch * d.n_kv_heads * d.kv_len * d.head_dim / 4, clear_grid = (n4 + 255) / 256;
  if (s.clear && !launch_fits(clear_grid, 256)) return fail(LOONG_E_UNSUPPORTED, "backward grid too large");
  // ---- the launch fits: from here on work is enqueued
  if (before)
    if (int rc = launch_prologue(d, *before, stream)) return rc;
  if (s.clear) {
    for (int t = 0; t < n; ++t)
      zero_kernel<<<dim3((unsigned)clear_grid), dim3(256), 0, st>>>(n4, reinterpret_cast<float4*>(dk[t]), reinterpret_cast<float4*>(dv[t]));
    if (int rc = check_launch("loong_attn_step_bwd (clear dk/dv)")) return rc;
  }
  if (!s.do_kv && !s.do_q) return LOONG_OK;
  if (d.dtype == LOONG_FP16) return pick_cfg<Fp16>(s, plan.tab, d.head_dim, plan.ks, dev.cus, st);
  return pick_cfg<Bf16>(s, plan.tab, d.head_dim, plan.ks, dev.cus, st);
}

// (all its keys counted as seen, and as many workgroups as make_work_map may add)
int64_t bwd_steps_that_fit_bf16(const loong_step_desc& d, const StepGeom& g) {
  const int64_t per_step = (int64_t)g.nk * ((g.k[0].len + kBwdBN - 1) / kBwdBN) * d.n_kv_heads * d.batch;
  return std::max<int64_t>((kMaxGrid - 8) / std::max<int64_t>(per_step, 1), 1);
}

}  // namespace loong
