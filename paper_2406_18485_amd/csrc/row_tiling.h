// Host-side choice of the work split for the kernels whose workgroups own query rows
// (the forward step and the dQ pass of the backward step).  A workgroup has eight waves =
// NRB row blocks of 32 rows x KS key splits; GS heads of one kv group share a workgroup.
#pragma once
#include <algorithm>
#include <cmath>

#include "loong_internal.h"

namespace loong {

constexpr int kRowWaves = 8;

// heads of one kv group stacked in a workgroup: the largest power of two that divides the
// group size and fits the row blocks
inline int pick_gs(int G, int nrb) {
  for (int gs = 8; gs >= 1; gs >>= 1)
    if (G % gs == 0 && gs <= nrb) return gs;
  return 1;
}

// does q segment a see any key in this step?
inline bool segment_sees_keys(const StepGeom& g, int a) {
  for (int kb = 0; kb < g.nk; ++kb)
    if (g.cls[a][kb] != LOONG_SKIP && g.k[kb].len > 0) return true;
  return false;
}

// number of q tiles of height bmh (rows per head) that have visible keys
inline int64_t busy_row_tiles(const StepGeom& g, int bmh) {
  int64_t n = 0;
  for (int a = 0; a < g.nq; ++a)
    if (segment_sees_keys(g, a)) n += (g.q[a].len + bmh - 1) / bmh;
  return n;
}

// Key splits: more splits give more workgroups, but each workgroup streams the whole visible
// K/V of its head through its own LDS and keeps fewer rows per staged tile, so the smallest
// split that puts a workgroup on (nearly) every compute unit is taken (measured on
// 32K..1M-token shapes: one more split than that is always slower, one fewer leaves units idle).
// `forced` (1, 2 or 4, from the descriptor's flags) overrides the choice; `cus` is the device's
// number of compute units.
inline int pick_key_splits(const StepGeom& g, int G, int Hq, int B, int forced, int cus) {
  if (forced == 1 || forced == 2 || forced == 4) return forced;
  // a step with a diagonal block has tiles of very different length: two workgroups per unit,
  // longest first, even them out
  bool diag = false;
  for (int a = 0; a < g.nq; ++a)
    for (int kb = 0; kb < g.nk; ++kb) diag |= g.cls[a][kb] == LOONG_DIAG;
  const int64_t want = (diag ? 2 : 1) * (int64_t)cus * 7 / 8;
  const int ks_opts[3] = {1, 2, 4};
  for (int i = 0; i < 3; ++i) {
    const int nrb = kRowWaves / ks_opts[i], gs = pick_gs(G, nrb);
    const int64_t n = busy_row_tiles(g, 32 * nrb / gs) * (Hq / gs) * B;
    if (n >= want) return ks_opts[i];
  }
  return 4;
}

// Key splits of a forward step.  Without a diagonal block all its workgroups are equally long, so a launch
// takes as many rounds as its workgroups fill the chip, and a round costs nearly the same whether it is
// full or not: fixed + per key (ns; measured at 1000 and 4096 keys with 1, 2, 4 splits).  At head_dim 64 two
// workgroups share a unit and a pair of rounds costs less than two.  The split with the least time is taken
// (ties: the taller tiles, which read K and V less often).  Against the smallest split that nearly fills the chip, 8 heads,
// 4096 keys, head_dim 128: 2304 rows 79.7 -> 66.7 us, 3000 rows 79.1 -> 67.8, 4500 rows 134 -> 106, 9000 rows 223 -> 209.
inline int pick_fwd_key_splits(const StepGeom& g, int G, int Hq, int B, int head_dim, int forced, int cus) {
  bool diag = false;
  double keys = 0;
  for (int a = 0; a < g.nq; ++a) {
    for (int kb = 0; kb < g.nk; ++kb) diag |= g.cls[a][kb] == LOONG_DIAG;
    keys = std::max(keys, keys_of_rows(g, a));
  }
  if (forced || diag) return pick_key_splits(g, G, Hq, B, forced, cus);
  struct Cost { double fixed, per_key; };
  const Cost one128[3] = {{9400, 23.1}, {9300, 13.95}, {8000, 7.8}};
  const Cost one64[3] = {{6500, 17.1}, {6500, 11.0}, {5800, 5.9}}, two64[3] = {{12200, 26.8}, {9900, 18.1}, {7800, 9.7}};
  int best = 4;
  double least = INFINITY;
  for (int i = 2; i >= 0; --i) {
    const int ks = 1 << i, nrb = kRowWaves / ks, gs = pick_gs(G, nrb);
    const int64_t n = busy_row_tiles(g, 32 * nrb / gs) * (Hq / gs) * B, rounds = (n + cus - 1) / cus;
    auto time = [&](const Cost& c) { return c.fixed + c.per_key * keys; };
    const double t = head_dim == 64 ? (rounds / 2) * time(two64[i]) + (rounds % 2) * time(one64[i]) : rounds * time(one128[i]);
    if (t <= least) { least = t; best = ks; }
  }
  return best;
}

// Placement of the row tiles of a launch with NRB row blocks per workgroup.  With
// `list_blind` false, q segments that see no key in this step get no tiles at all: the work
// list then holds busy tiles only, and cutting it into eight equal ranges (one per XCD)
// balances the chip.
struct RowTiling {
  int GS, ntile[2], tiles_total, hgroups;
  int64_t total_wg;
};

inline RowTiling make_row_tiling(const StepGeom& g, int G, int Hq, int B, int nrb, bool list_blind) {
  RowTiling t{};
  t.GS = pick_gs(G, nrb);
  const int bmh = 32 * nrb / t.GS;
  for (int a = 0; a < 2; ++a) {
    t.ntile[a] = a < g.nq && (list_blind || segment_sees_keys(g, a)) ? (g.q[a].len + bmh - 1) / bmh : 0;
    t.tiles_total += t.ntile[a];
  }
  t.hgroups = Hq / t.GS;
  t.total_wg = (int64_t)t.tiles_total * t.hgroups * B;
  return t;
}

}  // namespace loong
