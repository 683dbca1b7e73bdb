// fp32-storage kernels of the ring step on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 sums, nothing rounded to a shorter type).
//
// What bounds them: the shapes this storage type is used at are small (a correctness run, a first try), so a
// step is a few microseconds of dependent latencies (load, product, exponential, product, store), not a rate.
// Hence 16-row tiles (many workgroups from few rows), operands straight from global memory into
// registers (no LDS, no barrier in the loop), and the loop of a tile dealt out over the waves of its
// workgroup, which add up their parts through LDS once, in wave order.
//
// Layout.  Lane l = 16 g + i of a wave.  The instruction takes A[i][k = g], B[k = g][i] and gives
// D[4 g + v][i], v = 0..3.  Two kinds of fragment make every access 16 bytes per lane:
//   row fragment   lane holds x[row i][16 m + 4 g .. +3]: slice (m, v) of a contraction over columns takes
//                  component v, i.e. columns {16 m + 4 g + v}; A and B agree, so the order does not matter
//   column fragment lane holds x[row 4 g + v][VW i .. +VW-1] (+ 16 VW per strip): a contraction over rows
//                  takes rows {4 g + v} in slice v, which is register v of the D tile of the first
//                  product, and block (strip, b) of the result takes component b: its row 4 g + r is
//                  column strip 16 VW + VW (4 g + r) + b, so a lane ends with 4 VW consecutive columns of its row
// The first products are transposed (S^T = K Q^T; S = Q K^T where keys are owned), so their D tile is the B
// operand of the second product without any exchange.
//
// Against one wave per row with vector multiply-adds (a pass of a replay): 2 x 256 rows, 4 x 256 keys, d = 64,
// forward and backward 580 -> 102 us; 16 heads x 1024 rows, 2 x 1024 keys, d = 128 forward 1914 -> 130 us,
// backward 8494 -> 464 us.  Head dimensions other than 32, 64 and 128 take the kernels of 128 with the pieces past
// the end masked: up to 3.5 times the products (head_dim 36), the 16-row forward holds 31 registers of a lane in memory,
// the backward runs one wave per SIMD; still below one wave per row (4 heads x 500 rows, head_dim 36, forward 82.1 -> 25.5 us,
// backward 198 -> 37.8).  The distance from 64-bit results fell too (gradients 5.0e-7 -> 4.3e-7 relative).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_utils.h"
#include "loong_internal.h"
#include "step_table.h"
#include "work_map.h"

namespace loong {
namespace {

struct F32Params {
  const float *q, *d_o, *lse_in, *delta;
  float *out, *lse, *dq;
  float* stored;          // forward, or NULL: `out`, contiguous, is also copied here
  int B, Hq, Hkv, G, d, q_len, kv_len;
  int64_t qs[3], ks[3], os[3];
  StepGeom g;
  float scale;
  int fuse;
  uint16_t overwrite, accumulate;
  int rtile[2], rtiles;   // row tiles per q segment, in all
  int ktile[2], ktiles;   // key tiles per k segment, in all
  WorkMap rmap, kmap;     // units = batch x q heads (kv heads), items = row (key) tiles
};

// The micro-steps of a backward launch (a pass of 4 steps, 2 heads x 256 rows, d = 64, with its forward: 81 us
// with a launch per step, 61 with one): they share the geometry but for the block classes (two bits each:
// q segment 0 x key segments 0, 1, then q segment 1).
// (On a line of the scalar cache: eight bytes off, the backward of 1 row x 2048 keys, d = 128, takes 90 us, not 86.)
struct alignas(64) F32Run {
  const float *k[kMaxSteps], *v[kMaxSteps];
  float *dk[kMaxSteps], *dv[kMaxSteps];
  uint32_t cls[kMaxSteps];
  int n;
};
uint32_t classes(const StepGeom& g) { return g.cls[0][0] | g.cls[0][1] << 2 | g.cls[1][0] << 4 | g.cls[1][1] << 6; }
// The micro-steps of a forward launch: a step is some 8 us of latencies, of which the launch, the first loads and the way of
// the running rows through memory are the larger part (4 steps of 2 heads x 256 rows, d = 64: 38 -> 22 us).  A single step
// has a kernel without the search for the next one (256 rows, 2 heads on 1, d = 64: 8.9 -> 8.2 us, 2048 x 512 x 6 27.0 -> 24.9),
// whose arguments take no more lines of the scalar cache than it needs (one more is 0.3 us).
template <int N>
struct F32Steps {
  const float *k[N], *v[N];
  uint32_t cls[N];
  int n;
};
template <>
struct F32Steps<1> {
  const float *k, *v;
};
__device__ __forceinline__ StepGeom with_classes(const StepGeom& g, uint32_t c) {
  StepGeom x = g;
  x.cls[0][0] = c & 3; x.cls[0][1] = c >> 2 & 3; x.cls[1][0] = c >> 4 & 3; x.cls[1][1] = c >> 6 & 3;
  return x;
}

constexpr int kT = 16;           // rows / keys of a tile
constexpr int kMaxWaves = 8;     // waves that share a tile's loop
// (four waves at d = 128: they need more than the 256 registers that eight leave each; at d = 64 eight are
// better than four, 233 against 287 us a pass of 16 heads x 1024 rows)
constexpr int max_bwd_waves(int np) { return np == 128 ? 4 : kMaxWaves; }

__device__ __forceinline__ floatx4_t mfma16(float a, float b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// maximum / sum over the four lanes 16 g + i, g = 0..3
__device__ __forceinline__ float max_over_groups(float x) {
  const uintx2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_with_other_half(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_over_groups(float x) {
  const uintx2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return sum_with_other_half(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// NP: head_dim rounded up to the instruction's blocks; EXACT: head_dim == NP
template <int NP, bool EXACT>
struct Frag {
  static constexpr int NM = NP / 16;            // 16-byte pieces per lane of a row fragment; blocks of a result
  static constexpr int VW = NP == 32 ? 2 : 4;   // columns per lane and strip of a column fragment
  static constexpr int NS = NP / (16 * VW);     // strips
  typedef float vec_t __attribute__((ext_vector_type(VW)));
  struct Row { floatx4_t x[NM]; };
  struct Col { vec_t x[4][NS]; };
  struct Acc { floatx4_t x[NM]; };              // block strip * VW + b

  // row fragment of the row at `row` (head_dim d)
  static __device__ __forceinline__ Row load_row(const float* row, int g, int d) {
    Row f;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int c = 16 * m + 4 * g;
      if constexpr (EXACT) {
        f.x[m] = *reinterpret_cast<const floatx4_t*>(row + c);
      } else {  // pieces past the end contribute nothing
        const floatx4_t y = *reinterpret_cast<const floatx4_t*>(row + min(c, d - 4));
        f.x[m] = c < d ? y : floatx4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
    return f;
  }
  // column fragment of rows `first` + 4 g + v, the ones past `last` repeating it
  static __device__ __forceinline__ Col load_col(const float* base, int64_t stride, int first, int last, int i, int g, int d) {
    Col f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* row = base + (int64_t)min(first + 4 * g + v, last) * stride;
#pragma unroll
      for (int s = 0; s < NS; ++s) {  // (columns past the end: block rows that are never stored)
        const int c = 16 * VW * s + VW * i;
        f.x[v][s] = *reinterpret_cast<const vec_t*>(row + (EXACT ? c : min(c, d - VW)));
      }
    }
    return f;
  }
  // D = A B^T over the columns, two chains (the additions of one wait for each other)
  static __device__ __forceinline__ floatx4_t rows_product(const Row& a, const Row& b) {
    floatx4_t d0 = {0.f, 0.f, 0.f, 0.f}, d1 = d0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      d0 = mfma16(a.x[m][0], b.x[m][0], d0); d1 = mfma16(a.x[m][1], b.x[m][1], d1);
      d0 = mfma16(a.x[m][2], b.x[m][2], d0); d1 = mfma16(a.x[m][3], b.x[m][3], d1);
    }
    return d0 + d1;
  }
  // acc += A^T w over the 16 rows of A, w = D tile
  static __device__ __forceinline__ void cols_product(Acc& acc, const Col& a, floatx4_t w) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NM; ++n) acc.x[n] = mfma16(a.x[v][n / VW][n % VW], w[v], acc.x[n]);
  }
  // The same where some pairs are masked: a weight of zero must keep a row out whatever its values are, but
  // the matrix instruction multiplies (0 x infinity).  `ok`: bit v = pair (row 4 g + v, lane's column) takes part.
  static __device__ __forceinline__ void cols_product_masked(Acc& acc, const Col& a, floatx4_t w, int ok, const float* base,
                                                             int64_t stride, int first, int last, int i, int g, int d) {
    float z = 0.f;  // NaN if any element is not finite
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < NM; ++n) z = fmaf(a.x[v][n / VW][n % VW], 0.f, z);
    if (__builtin_amdgcn_ballot_w64(z != z) == 0) return cols_product(acc, a, w);
#pragma unroll 1
    for (int t = 0; t < kT; ++t) {
      const int v = t & 3, from = (t >> 2) * 16 + i;
      const float wt = __shfl(v == 0 ? w[0] : v == 1 ? w[1] : v == 2 ? w[2] : w[3], from, 64);
      const int okt = __shfl(ok, from, 64) >> v & 1;
      const float* row = base + (int64_t)min(first + t, last) * stride;
#pragma unroll
      for (int n = 0; n < NM; ++n) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = row[EXACT ? column(n, r, g) : min(column(n, r, g), d - 1)];
          acc.x[n][r] = okt ? fmaf(wt, x, acc.x[n][r]) : acc.x[n][r];
        }
      }
    }
  }
  static __device__ __forceinline__ int column(int n, int r, int g) { return 16 * VW * (n / VW) + VW * (4 * g + r) + n % VW; }
  // piece p of the lane's columns: four consecutive ones, starting at piece_col(p)
  static __device__ __forceinline__ int piece_col(int p, int g) { return 16 * VW * (p / VW) + 4 * VW * g + 4 * (p % VW); }
  static __device__ __forceinline__ floatx4_t piece(const Acc& a, int p) {
    floatx4_t x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int in_strip = 4 * (p % VW) + e;   // column inside the lane's 4 VW: VW r + b
      x[e] = a.x[(p / VW) * VW + in_strip % VW][in_strip / VW];
    }
    return x;
  }
  static __device__ __forceinline__ void set_piece(Acc& a, int p, floatx4_t x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int in_strip = 4 * (p % VW) + e;
      a.x[(p / VW) * VW + in_strip % VW][in_strip / VW] = x[e];
    }
  }
  static __device__ __forceinline__ Acc zero() {
    Acc a;
#pragma unroll
    for (int n = 0; n < NM; ++n) a.x[n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    return a;
  }
};

// The visible tiles of a row tile (key tiles) or of a key tile (row tiles of one head): per segment a
// first tile and a count, walked as one list.
struct TileList {
  int n0, total, first0, first1, len0, len1, start0, start1;
  bool diag0, diag1;
  struct Tile { int j0, len, start; bool diag; };
  __device__ __forceinline__ Tile at(int t) const {
    const bool s1 = t >= n0;
    return Tile{((s1 ? first1 + t - n0 : first0 + t)) * kT, s1 ? len1 : len0, s1 ? start1 : start0, s1 ? diag1 : diag0};
  }
};
__device__ __forceinline__ TileList keys_of_rows(const StepGeom& g, int qa, int last_row) {
  const int c0 = qa ? g.cls[1][0] : g.cls[0][0], c1 = g.nk > 1 ? (qa ? g.cls[1][1] : g.cls[0][1]) : LOONG_SKIP;
  TileList l{};
  l.len0 = g.k[0].len; l.len1 = g.nk > 1 ? g.k[1].len : 0;
  l.start0 = g.k[0].start; l.start1 = g.nk > 1 ? g.k[1].start : 0;
  l.diag0 = c0 == LOONG_DIAG; l.diag1 = c1 == LOONG_DIAG;
  const int e0 = c0 == LOONG_SKIP ? 0 : l.diag0 ? min(l.len0, last_row + 1) : l.len0;
  const int e1 = c1 == LOONG_SKIP ? 0 : l.diag1 ? min(l.len1, last_row + 1) : l.len1;
  l.n0 = (e0 + kT - 1) / kT;
  l.total = l.n0 + (e1 + kT - 1) / kT;
  return l;
}
__device__ __forceinline__ TileList rows_of_keys(const StepGeom& g, int kb, int first_key) {
  const int c0 = kb ? g.cls[0][1] : g.cls[0][0], c1 = g.nq > 1 ? (kb ? g.cls[1][1] : g.cls[1][0]) : LOONG_SKIP;
  TileList l{};
  l.len0 = g.q[0].len; l.len1 = g.nq > 1 ? g.q[1].len : 0;
  l.start0 = g.q[0].start; l.start1 = g.nq > 1 ? g.q[1].start : 0;
  l.diag0 = c0 == LOONG_DIAG; l.diag1 = c1 == LOONG_DIAG;
  const int t0 = (l.len0 + kT - 1) / kT, t1 = (l.len1 + kT - 1) / kT;
  l.first0 = l.diag0 ? min(first_key / kT, t0) : 0;
  l.first1 = l.diag1 ? min(first_key / kT, t1) : 0;
  l.n0 = c0 == LOONG_SKIP ? 0 : t0 - l.first0;
  l.total = l.n0 + (c1 == LOONG_SKIP ? 0 : t1 - l.first1);
  return l;
}

// Sum of the waves' accumulators, in wave order; afterwards wave w holds the pieces p with p % waves == w.
template <class F>
__device__ __forceinline__ void add_waves(typename F::Acc& a, floatx4_t* slots, int wave, int waves, int lane) {
#pragma unroll
  for (int p = 0; p < F::NM; ++p) slots[(wave * F::NM + p) * 64 + lane] = F::piece(a, p);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < F::NM; ++p)
    if (p % waves == wave) {
      floatx4_t x = slots[p * 64 + lane];
      for (int w = 1; w < waves; ++w) x += slots[(w * F::NM + p) * 64 + lane];
      F::set_piece(a, p, x);
    }
}

// ---- forward: RB x 16 query rows per workgroup (RB = 2 where rows are many: half the reads of K and V), over the
// launch's steps.  Between two steps the running result goes through LDS as it would go through memory: the same bits.
template <int NP, bool EXACT, int RB, int N>
__global__ __launch_bounds__(kMaxWaves * 64 / RB) void fwd_f32_kernel(const F32Params p, const F32Steps<N> steps) {
  using F = Frag<NP, EXACT>;
  constexpr int NM = F::NM;
  __shared__ floatx4_t slots[kMaxWaves * (NM + 1) * 64];
  // The running result between two steps goes where the first wave's part was, which the thread that forms it alone reads.  (Padded
  // 16-row form, which runs out of registers: apart; they are given out better then, head_dim 100, 100 rows x 4000 keys x 2 heads 118 us
  // against 131.)
  constexpr bool APART = !EXACT && RB == 1;
  __shared__ floatx4_t apart[APART ? NM * 64 : 1];
  floatx4_t* const state = APART ? apart : slots;
  constexpr int STATE_RB = APART ? NM : NM + 1;
  int bh, rank;
  if (!decode_work(p.rmap, blockIdx.x, bh, rank)) return;
  const int tt = p.rtiles - 1 - rank;  // late rows see more keys: first
  const int b = bh / p.Hq, h = bh - b * p.Hq, hk = h / p.G;
  const int qa = tt >= p.rtile[0] ? 1 : 0;
  const int row0 = (qa ? tt - p.rtile[0] : tt) * kT * RB;
  const Segment qs = qa ? p.g.q[1] : p.g.q[0];
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;

  // the next step in which the last of these rows sees a key
  TileList keys{};
  const float *kbase = nullptr, *vbase = nullptr;
  int step = -1;
  auto next_step = [&] {
    if constexpr (N == 1) {
      if (++step) return false;
      keys = keys_of_rows(p.g, qa, min(row0 + kT * RB, qs.len) - 1);
      kbase = steps.k + b * p.ks[0] + hk * p.ks[1];
      vbase = steps.v + b * p.ks[0] + hk * p.ks[1];
      return keys.total > 0;
    } else {
      for (++step; step < steps.n; ++step) {
        keys = keys_of_rows(with_classes(p.g, steps.cls[step]), qa, min(row0 + kT * RB, qs.len) - 1);
        if (keys.total == 0) continue;
        kbase = steps.k[step] + b * p.ks[0] + hk * p.ks[1];
        vbase = steps.v[step] + b * p.ks[0] + hk * p.ks[1];
        return true;
      }
      return false;
    }
  };
  bool more = next_step();
  if (!more && p.fuse && !p.stored) return;  // running result untouched

  typename F::Row qf[RB], kf;
  typename F::Acc o[RB];
  float m[RB], l[RB];
  int64_t orow[RB];
  float* lse_p[RB];
  auto load_k = [&](int t) {
    const TileList::Tile tl = keys.at(min(t, keys.total - 1));
    return F::load_row(kbase + (int64_t)(tl.start + min(tl.j0 + i, tl.len - 1)) * p.ks[2], g, p.d);
  };
  if (more && wave < keys.total) kf = load_k(wave);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = qs.start + min(row0 + rb * kT + i, qs.len - 1);
    qf[rb] = F::load_row(p.q + b * p.qs[0] + h * p.qs[1] + (int64_t)row * p.qs[2], g, p.d);
    orow[rb] = b * p.os[0] + h * p.os[1] + (int64_t)row * p.os[2];
    lse_p[rb] = p.lse + ((int64_t)b * p.Hq + h) * p.q_len + row;
    o[rb] = F::zero();
    m[rb] = -INFINITY; l[rb] = 0.f;
    if (p.fuse && wave == 0) {  // the first wave starts from the running result
      const float prev = *lse_p[rb];
      floatx4_t x[NM];
#pragma unroll
      for (int pc = 0; pc < NM; ++pc)
        x[pc] = *reinterpret_cast<const floatx4_t*>(p.out + orow[rb] + (EXACT ? F::piece_col(pc, g) : min(F::piece_col(pc, g), p.d - 4)));
      if (prev != -INFINITY) {
        m[rb] = prev * kLog2e;
        l[rb] = g == 0 ? 1.f : 0.f;
#pragma unroll
        for (int pc = 0; pc < NM; ++pc) F::set_piece(o[rb], pc, x[pc]);
      }
      if (!more && row0 + rb * kT + i < qs.len) {  // nothing visible in any step: the copy alone
#pragma unroll
        for (int pc = 0; pc < NM; ++pc)
          if (EXACT || F::piece_col(pc, g) < p.d) *reinterpret_cast<floatx4_t*>(p.stored + orow[rb] + F::piece_col(pc, g)) = x[pc];
      }
    }
  }
  if (!more && p.fuse) return;
  const float c = p.scale * kLog2e;
  for (;;) {
  for (int t = wave; t < keys.total; t += waves) {
    const TileList::Tile tl = keys.at(t);
    const float* vtile = vbase + (int64_t)tl.start * p.ks[2];
    const typename F::Col vf = F::load_col(vtile, p.ks[2], tl.j0, tl.len - 1, i, g, p.d);
    const typename F::Row kn = load_k(t + waves);
    __builtin_amdgcn_sched_barrier(0);  // requested before the products that hide them
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int off = row0 + rb * kT + i;
      floatx4_t s = F::rows_product(kf, qf[rb]) * c;
      const bool masked = tl.j0 + kT > tl.len || (tl.diag && tl.j0 + kT - 1 > row0 + rb * kT);
      int ok = 15;
      if (masked) {
        ok = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int key = tl.j0 + 4 * g + v;
          const bool yes = key < tl.len && (!tl.diag || key <= off);
          ok |= yes ? 1 << v : 0;
          s[v] = yes ? s[v] : -INFINITY;
        }
      }
      const float mx = max_over_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
      if (__builtin_amdgcn_ballot_w64(mx > m[rb]) != 0) {
        const float m_new = fmaxf(m[rb], mx);
        const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(m[rb] - m_new);
        l[rb] *= alpha;
#pragma unroll
        for (int n = 0; n < NM; ++n) o[rb].x[n] *= alpha;
        m[rb] = m_new;
      }
      const float m_use = m[rb] == -INFINITY ? 0.f : m[rb];
      floatx4_t w;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        w[v] = fast_exp2(s[v] - m_use);
        l[rb] += w[v];
      }
      if (masked) F::cols_product_masked(o[rb], vf, w, ok, vtile, p.ks[2], tl.j0, tl.len - 1, i, g, p.d);
      else F::cols_product(o[rb], vf, w);
    }
    kf = kn;
  }

  // ---- the waves' parts: common maximum, weights, sum in wave order
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    floatx4_t* mine = slots + (wave * RB + rb) * (NM + 1) * 64 + lane;
#pragma unroll
    for (int pc = 0; pc < NM; ++pc) mine[pc * 64] = F::piece(o[rb], pc);
    mine[NM * 64] = floatx4_t{m[rb], l[rb], 0.f, 0.f};
  }
  __syncthreads();
  more = next_step();
  if (more && wave < keys.total) kf = load_k(wave);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const floatx4_t* part = slots + rb * (NM + 1) * 64 + lane;
    const int step_w = RB * (NM + 1) * 64;
    float m_all = -INFINITY, l_all = 0.f;
    for (int w = 0; w < waves; ++w) m_all = fmaxf(m_all, part[w * step_w + NM * 64][0]);
    const float m_ref = m_all == -INFINITY ? 0.f : m_all;
    for (int w = 0; w < waves; ++w) {
      const floatx4_t st = part[w * step_w + NM * 64];
      l_all += st[1] * fast_exp2(st[0] - m_ref);
    }
    const float l_tot = sum_over_groups(l_all);
    const float inv = l_tot != 0.f ? 1.f / l_tot : 0.f;
    const float lse = l_tot != 0.f ? fmaf(m_all, kLn2, fast_log2(l_tot) * kLn2) : -INFINITY;
    const bool row_ok = row0 + rb * kT + i < qs.len;
    for (int pc = wave; pc < NM; pc += waves) {
      floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < waves; ++w) acc += part[w * step_w + pc * 64] * fast_exp2(part[w * step_w + NM * 64][0] - m_ref);
      acc = acc * inv;
      if (more) {
        state[(rb * STATE_RB + pc) * 64 + lane] = acc;
      } else if (row_ok && (EXACT || F::piece_col(pc, g) < p.d)) {
        *reinterpret_cast<floatx4_t*>(p.out + orow[rb] + F::piece_col(pc, g)) = acc;
        if (p.stored) *reinterpret_cast<floatx4_t*>(p.stored + orow[rb] + F::piece_col(pc, g)) = acc;
      }
    }
    if (!more && row_ok && wave == 0 && g == 0) *lse_p[rb] = lse;
    // (the first wave goes on from the result, the others from nothing)
    const bool some = wave == 0 && lse != -INFINITY;
    m[rb] = some ? lse * kLog2e : -INFINITY;
    l[rb] = some && g == 0 ? 1.f : 0.f;
  }
  if (!more) return;
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    o[rb] = F::zero();
    if (wave == 0 && m[rb] != -INFINITY) {
#pragma unroll
      for (int pc = 0; pc < NM; ++pc) F::set_piece(o[rb], pc, state[(rb * STATE_RB + pc) * 64 + lane]);
    }
  }
  }
}

// ---- backward, row-owning half: the share of dQ of 16 query rows that the launch's steps have
template <int NP, bool EXACT>
__device__ __forceinline__ void dq_f32_body(const F32Params& p, const F32Run& run, uint32_t block, floatx4_t* slots) {
  using F = Frag<NP, EXACT>;
  constexpr int NM = F::NM;
  int bh, rank;
  if (!decode_work(p.rmap, block, bh, rank)) return;
  const int tt = p.rtiles - 1 - rank;
  const int b = bh / p.Hq, h = bh - b * p.Hq, hk = h / p.G;
  const int qa = tt >= p.rtile[0] ? 1 : 0;
  const int row0 = (qa ? tt - p.rtile[0] : tt) * kT;
  const Segment qs = qa ? p.g.q[1] : p.g.q[0];
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int off = row0 + i, row = qs.start + min(off, qs.len - 1);
  const int64_t q_off = b * p.qs[0] + h * p.qs[1] + (int64_t)row * p.qs[2];
  const typename F::Row qf = F::load_row(p.q + q_off, g, p.d), of = F::load_row(p.d_o + q_off, g, p.d);
  const int64_t srow = ((int64_t)b * p.Hq + h) * p.q_len + row;
  const float lse = p.lse_in[srow], dl = p.delta[srow];
  typename F::Acc acc = F::zero();
  bool any = false;
  for (int step = 0; step < run.n; ++step) {
    const TileList keys = keys_of_rows(with_classes(p.g, run.cls[step]), qa, min(row0 + kT, qs.len) - 1);
    any |= keys.total > 0;
    const float* kbase = run.k[step] + b * p.ks[0] + hk * p.ks[1];
    const float* vbase = run.v[step] + b * p.ks[0] + hk * p.ks[1];
    for (int t = wave; t < keys.total; t += waves) {
      const TileList::Tile tl = keys.at(t);
      const int64_t koff = (int64_t)(tl.start + min(tl.j0 + i, tl.len - 1)) * p.ks[2];
      const float* ktile = kbase + (int64_t)tl.start * p.ks[2];
      const typename F::Row kf = F::load_row(kbase + koff, g, p.d), vf = F::load_row(vbase + koff, g, p.d);
      const typename F::Col kc = F::load_col(ktile, p.ks[2], tl.j0, tl.len - 1, i, g, p.d);
      __builtin_amdgcn_sched_barrier(0);
      const floatx4_t s = F::rows_product(kf, qf), dp = F::rows_product(vf, of);
      const bool masked = tl.j0 + kT > tl.len || (tl.diag && tl.j0 + kT - 1 > row0);
      floatx4_t w;
      int ok = 0;
  #pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int key = tl.j0 + 4 * g + v;
        const bool yes = lse != -INFINITY && (!masked || (key < tl.len && (!tl.diag || key <= off)));
        ok |= yes ? 1 << v : 0;
        w[v] = yes ? fast_exp2(fmaf(s[v], p.scale, -lse) * kLog2e) * (dp[v] - dl) : 0.f;
      }
      if (masked) F::cols_product_masked(acc, kc, w, ok, ktile, p.ks[2], tl.j0, tl.len - 1, i, g, p.d);
      else F::cols_product(acc, kc, w);
    }
  }
  if (!any && !p.overwrite) return;
  add_waves<F>(acc, slots, wave, waves, lane);
  if (off >= qs.len || (lse == -INFINITY && !p.overwrite)) return;
  float* dst = p.dq + b * p.os[0] + h * p.os[1] + (int64_t)row * p.os[2];
#pragma unroll
  for (int pc = 0; pc < NM; ++pc)
    if (pc % waves == wave && (EXACT || F::piece_col(pc, g) < p.d)) {
      floatx4_t* at = reinterpret_cast<floatx4_t*>(dst + F::piece_col(pc, g));
      const floatx4_t x = F::piece(acc, pc) * p.scale;
      *at = p.overwrite ? x : *at + x;
    }
}

// ---- backward, key-owning half: dK and dV of 16 keys, over the rows of every head of the group
template <int NP, bool EXACT>
__device__ __forceinline__ void dkv_f32_body(const F32Params& p, const F32Run& run, int step, uint32_t block, floatx4_t* slots) {
  using F = Frag<NP, EXACT>;
  constexpr int NM = F::NM;
  int bhk, kt;  // key tiles in storage order see ever fewer rows
  if (!decode_work(p.kmap, block, bhk, kt)) return;
  const int b = bhk / p.Hkv, hk = bhk - b * p.Hkv;
  const int kb = kt >= p.ktile[0] ? 1 : 0;
  const int key0 = (kb ? kt - p.ktile[0] : kt) * kT;
  const Segment ks = kb ? p.g.k[1] : p.g.k[0];
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const TileList rows = rows_of_keys(with_classes(p.g, run.cls[step]), kb, key0);

  const int off = key0 + i, key = ks.start + min(off, ks.len - 1);
  const int64_t k_off = b * p.ks[0] + hk * p.ks[1] + (int64_t)key * p.ks[2];
  const typename F::Row kf = F::load_row(run.k[step] + k_off, g, p.d), vf = F::load_row(run.v[step] + k_off, g, p.d);
  typename F::Acc ak = F::zero(), av = F::zero();
  const int n = rows.total * p.G;
  for (int t = wave; t < n; t += waves) {
    const int gq = t / rows.total, h = hk * p.G + gq;
    const TileList::Tile tl = rows.at(t - gq * rows.total);
    const int64_t tile = b * p.qs[0] + h * p.qs[1] + (int64_t)tl.start * p.qs[2];
    const int64_t r = tile + (int64_t)min(tl.j0 + i, tl.len - 1) * p.qs[2];
    const int64_t srow = ((int64_t)b * p.Hq + h) * p.q_len + tl.start;
    const typename F::Row qf = F::load_row(p.q + r, g, p.d), of = F::load_row(p.d_o + r, g, p.d);
    float lse[4], dl[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ro = min(tl.j0 + 4 * g + v, tl.len - 1);
      lse[v] = p.lse_in[srow + ro]; dl[v] = p.delta[srow + ro];
    }
    __builtin_amdgcn_sched_barrier(0);
    const floatx4_t s = F::rows_product(qf, kf);
    const typename F::Col oc = F::load_col(p.d_o + tile, p.qs[2], tl.j0, tl.len - 1, i, g, p.d);  // (Q's registers are free)
    __builtin_amdgcn_sched_barrier(0);
    const floatx4_t dp = F::rows_product(of, vf);
    const typename F::Col qc = F::load_col(p.q + tile, p.qs[2], tl.j0, tl.len - 1, i, g, p.d);
    __builtin_amdgcn_sched_barrier(0);
    const bool masked = tl.j0 + kT > tl.len || (tl.diag && key0 + kT - 1 > tl.j0);
    floatx4_t w, e;
    int ok = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ro = tl.j0 + 4 * g + v;
      const bool yes = lse[v] != -INFINITY && (!masked || (ro < tl.len && (!tl.diag || off <= ro)));
      ok |= yes ? 1 << v : 0;
      w[v] = yes ? fast_exp2(fmaf(s[v], p.scale, -lse[v]) * kLog2e) : 0.f;
      e[v] = yes ? w[v] * (dp[v] - dl[v]) : 0.f;
    }
    if (masked) {
      F::cols_product_masked(av, oc, w, ok, p.d_o + tile, p.qs[2], tl.j0, tl.len - 1, i, g, p.d);
      F::cols_product_masked(ak, qc, e, ok, p.q + tile, p.qs[2], tl.j0, tl.len - 1, i, g, p.d);
    } else {
      F::cols_product(av, oc, w);
      F::cols_product(ak, qc, e);
    }
  }
  add_waves<F>(av, slots, wave, waves, lane);
  __syncthreads();
  add_waves<F>(ak, slots, wave, waves, lane);
  if (off >= ks.len) return;
  const int64_t dst = (((int64_t)b * p.Hkv + hk) * p.kv_len + key) * p.d;
#pragma unroll
  for (int pc = 0; pc < NM; ++pc)
    if (pc % waves == wave && (EXACT || F::piece_col(pc, g) < p.d)) {
      floatx4_t* at_k = reinterpret_cast<floatx4_t*>(run.dk[step] + dst + F::piece_col(pc, g));
      floatx4_t* at_v = reinterpret_cast<floatx4_t*>(run.dv[step] + dst + F::piece_col(pc, g));
      floatx4_t x = F::piece(ak, pc) * p.scale, y = F::piece(av, pc);
      if (p.accumulate) { x += *at_k; y += *at_v; }
      *at_k = x;
      *at_v = y;
    }
}

// Both halves of all steps in one launch, the longer workgroups first: the key-owning ones (`nk` per step) for one
// step, the `nq` row-owning ones, which walk over every step's keys, for several.
template <int NP, bool EXACT>
__global__ __launch_bounds__(max_bwd_waves(NP) * 64) void bwd_f32_kernel(const F32Params p, const F32Run run, uint32_t nk, uint32_t nq) {
  __shared__ floatx4_t slots[max_bwd_waves(NP) * Frag<NP, EXACT>::NM * 64];
  const bool rows_first = run.n > 1;
  const uint32_t n_first = rows_first ? nq : nk;
  const bool second = blockIdx.x >= n_first;
  const uint32_t block = blockIdx.x - (second ? n_first : 0u);
  if (second != rows_first) {
    dq_f32_body<NP, EXACT>(p, run, block, slots);
  } else {
    const uint32_t step = block / nk;
    dkv_f32_body<NP, EXACT>(p, run, (int)step, block - step * nk, slots);
  }
}

F32Params make_params(const loong_step_desc& d, const StepGeom& g) {
  F32Params p{};
  p.B = d.batch; p.Hq = d.n_q_heads; p.Hkv = d.n_kv_heads; p.G = d.n_q_heads / d.n_kv_heads;
  p.d = d.head_dim; p.q_len = d.q_len; p.kv_len = d.kv_len;
  for (int i = 0; i < 3; ++i) { p.qs[i] = d.q_stride[i]; p.ks[i] = d.kv_stride[i]; p.os[i] = d.o_stride[i]; }
  p.g = g; p.scale = d.softmax_scale;
  p.fuse = (d.flags & LOONG_FUSE_MERGE) != 0;
  p.overwrite = (d.flags & LOONG_OVERWRITE_DQ) != 0;
  p.accumulate = (d.flags & LOONG_ACCUM_DKV) != 0;
  return p;
}

int tiles(int len, int t) { return (len + t - 1) / t; }

void tile_rows(F32Params& p, int height) {
  p.rtiles = 0;
  for (int a = 0; a < 2; ++a) {
    p.rtile[a] = a < p.g.nq ? tiles(p.g.q[a].len, height) : 0;
    p.rtiles += p.rtile[a];
  }
  p.rmap = make_work_map((int64_t)p.B * p.Hq, p.rtiles);
}

// `most` waves share a tile's loop, fewer where the grid would hold more threads than a launch takes.
int pick_waves(int64_t workgroups, int most) {
  int w = most;
  while (w > 1 && workgroups * w * 64 >= (int64_t)1 << 32) w >>= 1;
  return w;
}

template <int NP, bool EXACT, int RB>
int launch_fwd_form(const F32Params& p, const F32Steps<kMaxSteps>& steps, int waves, hipStream_t st) {
  if (!launch_fits(p.rmap.grid, waves * 64)) return fail(LOONG_E_UNSUPPORTED, "fp32 path: forward grid too large");
  // (the padded 16-row form as compiled for a run is the faster one: 118 us against 142)
  if constexpr (EXACT || RB == 2) {
    if (steps.n == 1) {
      fwd_f32_kernel<NP, EXACT, RB, 1><<<dim3(p.rmap.grid), dim3(waves * 64), 0, st>>>(p, F32Steps<1>{steps.k[0], steps.v[0]});
      return check_launch("loong_attn_step_fwd (fp32)");
    }
  }
  fwd_f32_kernel<NP, EXACT, RB, kMaxSteps><<<dim3(p.rmap.grid), dim3(waves * 64), 0, st>>>(p, steps);
  return check_launch("loong_attn_step_fwd (fp32)");
}

template <int NP, bool EXACT>
int launch_fwd(F32Params& p, const F32Steps<kMaxSteps>& steps, int cus, hipStream_t st) {
  // 32-row workgroups where they still put two on every unit (16384 rows, d = 128, a pass of two steps: 131 us
  // against 156 with two waves per tile).  16-row ones share a tile among eight waves while that is at most two
  // waves per SIMD, else among four (4 heads x 600 rows, d = 128: 35 us with four, 41 with eight, 51 with two).
  tile_rows(p, 2 * kT);
  const int64_t wide = (int64_t)p.B * p.Hq * p.rtiles;
  if (wide >= 2 * cus) return launch_fwd_form<NP, EXACT, 2>(p, steps, pick_waves(p.rmap.grid, 4), st);
  tile_rows(p, kT);
  return launch_fwd_form<NP, EXACT, 1>(p, steps, pick_waves(p.rmap.grid, (int64_t)p.rmap.grid * kMaxWaves <= (int64_t)cus * 8 ? kMaxWaves : 4), st);
}

template <int NP, bool EXACT>
int launch_bwd(F32Params& p, const F32Run& run, bool do_dq, bool do_dkv, hipStream_t st) {
  tile_rows(p, kT);
  for (int a = 0; a < 2; ++a) {
    p.ktile[a] = a < p.g.nk ? tiles(p.g.k[a].len, kT) : 0;
    p.ktiles += p.ktile[a];
  }
  p.kmap = make_work_map((int64_t)p.B * p.Hkv, p.ktiles);
  const uint32_t nk = do_dkv ? p.kmap.grid : 0, nq = do_dq ? p.rmap.grid : 0;
  if (!launch_fits(nk, 64) || !launch_fits(nq, 64)) return fail(LOONG_E_UNSUPPORTED, "fp32 path: backward grid too large");
  const int64_t grid = (int64_t)nk * run.n + nq;
  if (grid * 64 < (int64_t)1 << 32) {
    const int w = pick_waves(grid, max_bwd_waves(NP));
    bwd_f32_kernel<NP, EXACT><<<dim3((unsigned)grid), dim3(w * 64), 0, st>>>(p, run, nk, nq);
    return check_launch("loong_attn_step_bwd (fp32)");
  }
  // more workgroups than one grid takes: step by step, half by half
  F32Run one{};
  one.n = 1;
  for (int t = 0; t < run.n; ++t) {
    one.k[0] = run.k[t]; one.v[0] = run.v[t]; one.dk[0] = run.dk[t]; one.dv[0] = run.dv[t]; one.cls[0] = run.cls[t];
    if (nk) bwd_f32_kernel<NP, EXACT><<<dim3(nk), dim3(pick_waves(nk, max_bwd_waves(NP)) * 64), 0, st>>>(p, one, nk, 0);
    if (nq) bwd_f32_kernel<NP, EXACT><<<dim3(nq), dim3(pick_waves(nq, max_bwd_waves(NP)) * 64), 0, st>>>(p, one, 0, nq);
    p.overwrite = 0;
  }
  return check_launch("loong_attn_step_bwd (fp32)");
}

}  // namespace

int launch_fwd_f32(const loong_step_desc* descs, int n, const void* q, const void* const* k, const void* const* v,
                   float* out, float* lse, void* stored, void* stream) {
  const loong_step_desc& d = descs[0];
  const int64_t rows = (int64_t)d.batch * d.n_q_heads * d.q_len;
  if (rows == 0) return LOONG_OK;
  if (rows > 0x7fffffff) return fail(LOONG_E_UNSUPPORTED, "fp32 path: more than 2^31-1 query rows");
  DeviceFacts dev;
  if (int rc = device_facts(&dev)) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  StepGeom g;
  if (int rc = check_step(&descs[0], &g)) return rc;
  F32Params p = make_params(d, g);
  p.q = (const float*)q; p.out = out; p.lse = lse;
  for (int t = 0; t < n;) {
    F32Steps<kMaxSteps> steps;
    steps.n = 0;
    for (; t < n && steps.n < kMaxSteps; ++t, ++steps.n) {
      if (int rc = check_step(&descs[t], &p.g)) return rc;
      steps.k[steps.n] = (const float*)k[t]; steps.v[steps.n] = (const float*)v[t];
      steps.cls[steps.n] = classes(p.g);
    }
    p.stored = t == n ? (float*)stored : nullptr;
    if (int rc = d.head_dim == 32    ? launch_fwd<32, true>(p, steps, dev.cus, st)
                 : d.head_dim == 64  ? launch_fwd<64, true>(p, steps, dev.cus, st)
                 : d.head_dim == 128 ? launch_fwd<128, true>(p, steps, dev.cus, st)
                                     : launch_fwd<128, false>(p, steps, dev.cus, st))
      return rc;
    p.fuse = 1;
  }
  return LOONG_OK;
}

int launch_bwd_f32(const loong_step_desc& d, const StepGeom* g, int n, const void* q, const void* const* k,
                   const void* const* v, const void* d_o, const float* lse, const float* delta, float* dq,
                   float* const* dk, float* const* dv, void* stream) {
  const int64_t qrows = (int64_t)d.batch * d.n_q_heads * d.q_len;
  const int64_t krows = (int64_t)d.batch * d.n_kv_heads * d.kv_len;
  if (qrows > 0x7fffffff || krows > 0x7fffffff)
    return fail(LOONG_E_UNSUPPORTED, "fp32 path: more than 2^31-1 rows");
  const bool do_dq = !(d.flags & LOONG_BWD_ONLY_DKV) && qrows > 0 && (krows > 0 || (d.flags & LOONG_OVERWRITE_DQ));
  const bool do_dkv = !(d.flags & LOONG_BWD_ONLY_DQ) && krows > 0;
  if (!do_dq && !do_dkv) return LOONG_OK;
  F32Params p = make_params(d, g[0]);
  p.q = (const float*)q; p.d_o = (const float*)d_o;
  p.lse_in = lse; p.delta = delta; p.dq = dq;
  F32Run run{};
  run.n = n;
  for (int t = 0; t < n; ++t) {
    run.k[t] = (const float*)k[t]; run.v[t] = (const float*)v[t];
    if (do_dkv) { run.dk[t] = dk[t]; run.dv[t] = dv[t]; }
    run.cls[t] = classes(g[t]);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (d.head_dim == 32) return launch_bwd<32, true>(p, run, do_dq, do_dkv, st);
  if (d.head_dim == 64) return launch_bwd<64, true>(p, run, do_dq, do_dkv, st);
  if (d.head_dim == 128) return launch_bwd<128, true>(p, run, do_dq, do_dkv, st);
  return launch_bwd<128, false>(p, run, do_dq, do_dkv, st);
}

}  // namespace loong
