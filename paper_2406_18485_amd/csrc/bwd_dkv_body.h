// Backward micro-step on the 16-bit matrix cores (element class E: bf16 or IEEE half; the text
// below says bf16 for both), dK/dV part: gradients of the visiting K/V chunk,
// recomputing the probabilities from the final softmax_lse (paper: Sec. 3.1 last paragraph;
// Sec. "Selective Checkpoint++").  This step's share of dQ comes from the row-owning half
// in bwd_dq_body.h.
//
// Work split.  A workgroup owns 128 keys of one kv head and walks over the 64-row query
// tiles of every q head of the group that can see them.  It has eight waves, two per SIMD:
// for each group of 32 keys a "P wave" and an "E wave" that sit on the same SIMD.
//   P wave   keeps the K rows (B operand) and the fp32 dV accumulator of its 32 keys:
//            S = Q K^T, P = exp2(S * scale * log2 e - LSE * log2 e), packed to bf16, handed
//            to its partner through LDS, then dV += P^T dO;
//   E wave   keeps the -V rows and the fp32 dK accumulator: T = delta - dO V^T straight out
//            of the matrix cores (the chain starts from C = delta), then E = P o T
//            (= -dS / scale), dK += E^T Q; dK is multiplied by -scale once, at the end.
// The E waves run one tile behind the P waves (P of tile t is consumed in the next iteration,
// from a double-buffered hand-over area; the query tiles stay in LDS for three iterations, the dO rows of the form for two
// workgroups per unit for two), so
// one workgroup barrier per tile suffices and neither role ever waits for the other.  The E
// waves, which have less element-wise work, also issue the staging loads.  A P wave's own
// dV += P^T dO of tile t also runs one iteration late, first thing after the barrier, from
// the P it kept in registers: the iteration then opens with matrix work on one wave of every
// SIMD while its partner issues the staging loads, instead of both starting with vector and
// memory instructions (2 % on the kernel, with the operand reads four matrix steps ahead).
// Splitting the roles halves the registers a wave must hold (so two waves fit a SIMD), and
// the two waves of a SIMD are in different kinds of work at any time: the vector issue port,
// which the matrix instructions share with the element-wise ones, is the unit that bounds
// this kernel, and every other instruction of one wave (LDS reads, waits, staging, scalar
// work) now hides behind the partner.
//
// Per query tile: Q, dO (row-major) and the rows' LSE and delta go from global memory
// straight into LDS, one tile ahead (head_dim 64: the LSE through a register of an E wave; two workgroups per unit: dO and delta an
// iteration later), with the 16-byte pieces of every row XOR-permuted so
// that both kinds of LDS read are free of bank conflicts: A operands of S / T are 16-byte
// reads of Q / dO rows (one key per lane, 16 query rows per 32x32 block in registers);
// the contractions over rows take P^T / E^T straight from registers as the A operand and
// transposing LDS reads of the same dO / Q tiles as the B operand.
#pragma once
#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "loong_internal.h"
#include "split_exchange.h"
#include "step_table.h"
#include "work_map.h"

namespace loong {
namespace {

struct DkvParams {
  const uint16_t *q, *d_o;
  const float *lse, *delta;
  int B, Hq, Hkv, G;
  int q_len, kv_len;
  int64_t qs[3], ks[3];
  int nq;
  Segment qseg[2];
  float scale, c;  // softmax scale; scale * log2(e)
  int accumulate;  // 1: the results are added to dk/dv instead of stored
  int nkt, kt_total;  // key tiles per half; of all seen halves
  int nsplit;      // workgroups that share the query loop of one key tile
  uint32_t* ws_cnt;  // nsplit > 1: counter per (batch, kv head, key tile), zero before and after the launch
  float* ws_part;    // nsplit > 1: partial dK/dV of every (key tile, split), in accumulator layout
  WorkMap map;     // units = batch x kv heads, items = key tiles x splits
};

constexpr int kBwdWaves = 8;            // 4 key groups x {P wave, E wave}
constexpr int kBwdBN = 128;             // keys per workgroup
constexpr int kBwdBM = 64;              // query rows per iteration

// (W: workgroups per unit the form is made for)
template <int D, int W>
struct BwdCfg {
  static constexpr int BM = kBwdBM, BN = kBwdBN;
  static constexpr int ROWB = D * 2;               // bytes per row of a Q / dO tile
  static constexpr int CH = D / 8;                 // 16-byte pieces per row
  static constexpr int RPI = 1024 / ROWB;          // rows filled by one wave-level load
  static constexpr int QT_B = BM * ROWB;           // bytes of a Q (or dO) tile
  static constexpr int LI = QT_B / 1024 / 4;       // loads per staging wave (the four E waves) per Q (or dO) tile
  // head_dim 64 can run two workgroups per unit (W = 2): one's prologue, epilogue and exchange of partial sums run beside the other's
  // loop, and four waves per SIMD leave the vector port idle less.  That takes at most 128 registers (operands requested three
  // steps ahead, not four) and half the LDS: the Q rows keep three stages (tile being staged, tile of the P waves, tile of the E
  // waves), but both roles use the dO rows of the E waves' tile only, so these are staged an iteration later, in two (LATE_O).
  // At head_dim 64 the P waves, whose exponentials weigh twice as much beside their matrix work, are the longer path, so the exponent
  // offsets of a tile's rows are formed once, by the E wave that fetches their LSE (OFFSETS).  dK/dV alone, one workgroup per
  // unit -> two -> with OFFSETS: 1500 rows x 4100 keys x 2 x 8 heads 116 -> 101 -> 87 us, 8192 x 8192 x 8 heads on 2
  // 298 -> 310 -> 275 (the last with twice the workgroups per query loop), 16384 x 16384 x 8 1165 -> 1040 -> 1023.  With OFFSETS in
  // one workgroup per unit ragged and diagonal tiles gain (800 rows, 4 heads on 1, 24.7 -> 22.6), long loops without a mask lose
  // (16384 x 2048 95 -> 98).
  // At head_dim 128 (registers for one workgroup) both cost: late dO 874 -> 905 us (16384 x 16384 x 4 heads), OFFSETS 516 -> 545
  // (8 steps of 2048 rows x 8 heads): the E waves' path is the longer one there.
  static constexpr bool LATE_O = W == 2, OFFSETS = D == 64;
  static constexpr int NSTAGE_Q = 3, NSTAGE_O = LATE_O ? 2 : 3;
  static constexpr int Q_STRIDE = (LATE_O ? 1 : 2) * (QT_B + BM * 4), O_STRIDE = Q_STRIDE;
  static constexpr int O_OFF = LATE_O ? NSTAGE_Q * Q_STRIDE : QT_B;            // first dO stage
  static constexpr int LSE_OFF = LATE_O ? QT_B : 2 * QT_B;                     // from the start of a Q stage
  static constexpr int DELTA_OFF = LATE_O ? QT_B : QT_B + BM * 4;              // from the start of a dO stage
  static constexpr int XCH_OFF = LATE_O ? O_OFF + NSTAGE_O * O_STRIDE : NSTAGE_Q * Q_STRIDE;
  static constexpr int XCH_B = 4 * 2 * 2 * 1024;   // P hand-over: 4 key groups x 2 blocks x 2 halves x 64 lanes x 16 B
  static constexpr int ROLE_OFF = XCH_OFF + 2 * XCH_B;  // shared loops: what arrive() said
  static constexpr int SMEM_BYTES = ROLE_OFF + 16;
  static_assert(LI >= 1 && LI * 1024 * 4 == QT_B, "tile must split evenly over the staging waves");
};

template <class E, int D, int W>
__device__ __forceinline__ void dkv_body(const StepTable& tab, const DkvParams& p, uint32_t block, unsigned char* smem) {
  using C = BwdCfg<D, W>;
  constexpr int BM = C::BM, BN = C::BN, ROWB = C::ROWB, CH = C::CH, LI = C::LI;
  constexpr int NKS = D / 16, NDB = D / 32;
  static_assert(BM == 64, "the pipeline below is written for two 32-row blocks per tile");

  // ---- which (batch, kv head, key tile, split)
  int bhk, rem;  // key tiles in storage order see ever fewer queries: that is the ranking
  if (!decode_work(p.map, block, bhk, rem)) return;
  const int kt = rem / p.nsplit, sp = rem - kt * p.nsplit;
  const int b = bhk / p.Hkv, hk = bhk - b * p.Hkv;
  const int half_idx = kt / p.nkt, koff0 = (kt - half_idx * p.nkt) * BN;
  const uint32_t entry0 = scalar_now(tab.first_half[0]), entry1 = scalar_now(tab.first_half[1]);
  uint32_t entry = half_idx == 1 ? entry1 : entry0;
  if (half_idx > 1) entry = tab.half[half_idx];
  const int step = entry_step(entry), klen = tab.klen, kstart = entry_half(entry) * klen;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const int kg = wave & 3;           // key group: keys koff0 + 32 kg ..
  const bool p_wave = wave < 4;      // waves kg and kg + 4 share a SIMD
  const bool p_wave_s = scalar_now(p_wave);  // (the same in a scalar register, where it chooses a pointer)
  const int my_koff = koff0 + 32 * kg + l32;
  const bool key_ok = my_koff < klen;
  const int64_t my_krow = kstart + min(my_koff, klen - 1);

  // ---- query tiles that can see this key tile: per q segment, tiles first .. first + cnt - 1
  // (per-segment facts in scalars: the loop never indexes the kernel arguments dynamically)
  const int clsq0 = entry_class(entry, 0), clsq1 = p.nq > 1 ? entry_class(entry, 1) : LOONG_SKIP;
  const int qlen0 = p.qseg[0].len, qlen1 = p.nq > 1 ? p.qseg[1].len : 0;
  const int qstart0 = p.qseg[0].start, qstart1 = p.nq > 1 ? p.qseg[1].start : 0;
  const int nt0 = (qlen0 + BM - 1) / BM, nt1 = (qlen1 + BM - 1) / BM;
  const int first0 = clsq0 == LOONG_DIAG ? min(koff0 / BM, nt0) : 0;
  const int first1 = clsq1 == LOONG_DIAG ? min(koff0 / BM, nt1) : 0;
  const int cnt0 = clsq0 == LOONG_SKIP ? 0 : nt0 - first0;
  const int cnt1 = clsq1 == LOONG_SKIP ? 0 : nt1 - first1;
  const int per_g = cnt0 + cnt1;
  const int n_it = per_g * p.G;
  const int it_begin = (int)((int64_t)n_it * sp / p.nsplit);
  const int it_end = (int)((int64_t)n_it * (sp + 1) / p.nsplit);
  // iteration -> (head of the group, tile inside the group's list); advanced without divisions
  struct Cursor { int gq, r; };
  auto advance = [&](Cursor& cu) {
    if (++cu.r == per_g) { cu.r = 0; ++cu.gq; }
  };
  auto decode = [&](const Cursor& cu, int& h, int& qa, int& i0) {
    qa = cu.r < cnt0 ? 0 : 1;
    i0 = (qa ? first1 + cu.r - cnt0 : first0 + cu.r) * BM;
    h = hk * p.G + cu.gq;
  };

  // ---- the wave's B operand: its K rows (P wave) or its V rows with the sign bits flipped
  // (E wave); row my_krow, columns 16 ks + 8 hh .. +7.  All of it is requested before any of it is used.
  bf16x8_t bfrag[NKS];
  {
    const uint16_t *kp = scalar_now(tab.step[0].k), *vp = scalar_now(tab.step[0].v);
    if (step) { kp = scalar_now(tab.step[step].k); vp = scalar_now(tab.step[step].v); }
    const uint16_t* row = (p_wave_s ? kp : vp) + b * p.ks[0] + hk * p.ks[1] + my_krow * p.ks[2];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) bfrag[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(row + ks * 16 + hh * 8));
  }
  // K comes with scale * log2 e folded in (rounded to 16 bits again): the score product then ends
  // in the exponent's units and its chains can start from the rows' offsets, which takes the
  // multiply-add per element off the vector port (4 % of the kernel).  The second rounding
  // changes P by less than rounding P itself to 16 bits does.
  if (p_wave_s) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) bfrag[ks] = scaled_fragment<E>(bfrag[ks], p.c);
  } else {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      uint4 x = __builtin_bit_cast(uint4, bfrag[ks]);
      x.x ^= 0x80008000u; x.y ^= 0x80008000u; x.z ^= 0x80008000u; x.w ^= 0x80008000u;
      bfrag[ks] = as_bf16x8(x);
    }
  }

  // ---- per-lane pieces of the staging and of the LDS reads
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  // direct loads (E waves): load i of staging wave kg fills LDS bytes [(kg + 4 i) * 1024, +1024) of a tile
  const int ld_row = kg * C::RPI + lane / CH;  // row inside the tile for i = 0; later loads add 4 * RPI rows
  const uint32_t ld_piece = (uint32_t)((lane % CH) ^ tile_swizzle<D>(ld_row)) * 16;
  const uint32_t q_rowbytes = (uint32_t)p.qs[2] * 2;  // validated: token stride < 2^24 elements
  uint32_t ld_off[LI];  // byte offset of this lane's piece from the tile's first row
#pragma unroll
  for (int i = 0; i < LI; ++i) ld_off[i] = (uint32_t)(ld_row + i * 4 * C::RPI) * q_rowbytes + ld_piece;
  // A operand of S / T: row l32 (+32 ib), pieces 2 ks + hh; transposing reads of a row-major tile: run of four rows starting
  // at 4 hh (+8 for the second run; +16 sl, +32 ib as constants), 16-column strip (lane >> 4) & 1 of block db
  uint32_t row_rd[NKS], tr_lo[NDB], tr_hi[NDB];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) row_rd[ks] = row_read_base<D>(lane) ^ row_read_xor(ks);
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    tr_lo[db] = tr_read_base<D>(lane) ^ tr_read_xor(db, 0);
    tr_hi[db] = (tr_read_base<D>(lane) ^ tr_read_xor(db, 1)) + 8 * ROWB;
  }
  // P hand-over slot of this key group: [block][half of the block's 16 elements][lane] x 16 bytes
  unsigned char* const xch = smem + C::XCH_OFF + kg * 4096 + lane * 16;

  floatx16_t acc[NDB];  // dV (P wave) or dK / -scale (E wave) of the wave's 32 keys
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;

  // ---- staging of one query tile by the E waves, global -> LDS: Q rows into the stage at byte `at_q`, dO rows and their
  // delta into the one at `at_o` (either may be left out); with OFFSETS the rows' LSE goes to a register of E wave 0
  float lse_ahead = 0.f;
  auto issue_tile = [&](const Cursor& cu, auto want_q, auto want_o, uint32_t at_q, uint32_t at_o) {
    if (p_wave) return;
    int h, qa, i0;
    decode(cu, h, qa, i0);
    const int qlen = qa ? qlen1 : qlen0, qstart = qa ? qstart1 : qstart0;
    const int last = qlen - 1 - i0;
    const int64_t tile_off = b * p.qs[0] + h * p.qs[1] + (int64_t)(qstart + i0) * p.qs[2];
    const unsigned char* qb = reinterpret_cast<const unsigned char*>(p.q + tile_off);
    const unsigned char* ob = reinterpret_cast<const unsigned char*>(p.d_o + tile_off);
    const uint32_t sq = smem_base + at_q, so = smem_base + at_o;
    if (last >= BM - 1) {
#pragma unroll
      for (int i = 0; i < LI; ++i) {
        if constexpr (want_q.value) load_to_lds_16(qb, ld_off[i], sq + (kg + 4 * i) * 1024);
        if constexpr (want_o.value) load_to_lds_16(ob, ld_off[i], so + (kg + 4 * i) * 1024);
      }
    } else {  // ragged end of a segment: rows past the last one repeat it
#pragma unroll
      for (int i = 0; i < LI; ++i) {
        const uint32_t off = (uint32_t)min(ld_row + i * 4 * C::RPI, last) * q_rowbytes + ld_piece;
        if constexpr (want_q.value) load_to_lds_16(qb, off, sq + (kg + 4 * i) * 1024);
        if constexpr (want_o.value) load_to_lds_16(ob, off, so + (kg + 4 * i) * 1024);
      }
    }
    const int64_t row = ((int64_t)b * p.Hq + h) * p.q_len + qstart + i0 + min(lane, last);
    if constexpr (C::OFFSETS) {
      if constexpr (want_q.value)
        if (kg == 0) lse_ahead = lane <= last ? p.lse[row] : -INFINITY;
      if constexpr (want_o.value)
        if (kg == 1) load_to_lds_4(p.delta + row, so + C::DELTA_OFF);
    } else {
      if (kg < 2) load_to_lds_4((kg ? p.delta : p.lse) + row, sq + C::LSE_OFF + kg * BM * 4);  // E wave 0: the LSE, E wave 1: delta
    }
  };
  // E wave 0, once the LSE of a staged tile is there: the exponent offsets its rows' score chains start from, -LSE log2 e, and -inf
  // (P = 0) for rows past the end of the segment and rows that saw no key in the whole attention (also where the lowest float says so)
  auto store_offsets = [&](int stage) {
    const float offset = lse_ahead * -kLog2e;
    if (C::OFFSETS && wave == 4)
      *reinterpret_cast<float*>(smem + stage * C::Q_STRIDE + C::LSE_OFF + lane * 4) = offset == INFINITY ? -INFINITY : offset;
  };
  constexpr std::true_type yes;
  constexpr std::false_type no;

  Cursor cur, nxt;
  cur.gq = it_begin / max(per_g, 1);
  cur.r = it_begin - cur.gq * per_g;
  nxt = cur;

  wait_vmcnt<0>();  // the K / V fragments are in: no counter wait of the compiler's lands in the loop
  if (it_begin < it_end) {
    if constexpr (C::LATE_O) issue_tile(cur, yes, no, 0, 0);
    else issue_tile(cur, yes, yes, 0, C::O_OFF);
  }
  if (!p_wave) wait_vmcnt<0>();
  store_offsets(0);

  // ---- the gradients of keys no query sees: the unit's workgroups clear a share each, from
  // the P waves (their stores have the first iteration to finish; as a launch of its own this cost
  // 5-7 us a step)
  if (p_wave && !p.accumulate)
    for (int z = tab.n_seen; z < tab.n_halves; ++z) {
      const uint32_t ze = z == 1 ? entry1 : tab.half[z];
      const int64_t off = (((int64_t)b * p.Hkv + hk) * p.kv_len + (int64_t)entry_half(ze) * klen) * D;
      float4* zk = reinterpret_cast<float4*>(tab.step[entry_step(ze)].dk + off);
      float4* zv = reinterpret_cast<float4*>(tab.step[entry_step(ze)].dv + off);
      const int64_t n4 = (int64_t)klen * (D / 4), stride = (int64_t)p.map.per_unit * 256;
      for (int64_t i = (int64_t)rem * 256 + tid; i < n4; i += stride) {
        zk[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        zv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }

  // P and E = P o T packed, two bf16 per word (elements 2 w, 2 w + 1 of block ib).  A P wave keeps
  // its P across the barrier: dV += P^T dO of tile t runs at the top of iteration t + 1.
  uint32_t w2[2][8];
  constexpr int PF = W == 2 ? 3 : 4;  // LDS operands are requested PF matrix steps ahead
  // Iteration j: the P waves work on tile j, the E waves on tile j - 1; the Q rows of tile j + 1 and the dO rows of
  // tile j are staged.
  int st_p = 0, st_e = 2, st_n = 1;  // LDS stages of the Q rows of tiles j, j - 1 and j + 1
  int so_e = 1, so_n = 0;            // and of the dO rows of tiles j - 1 and j
  for (int it = it_begin; it <= it_end && it_begin < it_end; ++it) {
    __syncthreads();  // tile `it` is in LDS, P of tile it - 1 is handed over, tile it - 2 is finished with
    if (it + 1 < it_end) {
      advance(nxt);
      if constexpr (C::LATE_O) issue_tile(nxt, yes, no, st_n * C::Q_STRIDE, 0);
      else issue_tile(nxt, yes, yes, st_n * C::Q_STRIDE, st_n * C::Q_STRIDE + C::O_OFF);
    }
    if constexpr (C::LATE_O)
      if (it < it_end) issue_tile(cur, no, yes, 0, C::O_OFF + so_n * C::O_STRIDE);
    const bool p_active = p_wave && it < it_end, e_active = !p_wave && it > it_begin;
    int h, qa, i0;
    decode(cur, h, qa, i0);
    const int qlen = qa ? qlen1 : qlen0;
    const bool isdiag = (qa ? clsq1 : clsq0) == LOONG_DIAG;
    const bool need_mask = (!C::OFFSETS && i0 + BM > qlen) || koff0 + BN > klen || (isdiag && i0 < koff0 + BN - 1);
    const unsigned char* Qt = smem + (p_wave ? st_p : st_e) * C::Q_STRIDE;
    const unsigned char* Ot = smem + C::O_OFF + (C::LATE_O ? so_e : st_e) * C::O_STRIDE;  // of tile j - 1
    const float* nl_s = reinterpret_cast<const float*>(Qt + C::LSE_OFF);
    const float* dl_s = reinterpret_cast<const float*>(Ot + C::DELTA_OFF);
    unsigned char* const xch_w = xch + ((it - it_begin) & 1) * C::XCH_B;        // P of tile `it`
    const unsigned char* const xch_r = xch + ((it - it_begin + 1) & 1) * C::XCH_B;  // P of tile it - 1

    // Block ib = rows 32 ib .. 32 ib + 31 of the tile; register v of an accumulator is row
    // acc_row(v, hh) of the block.
    floatx16_t st2[2];
    // 2 NKS matrix steps of S (P wave: Q rows, K fragments) or T (E wave: dO rows, -V fragments)
    // of both blocks, block 1 after block 0; `between(k)` is called after step k.
    auto rows_product = [&](const unsigned char* tile, auto&& between) {
      auto operand = [&](int k) {
        return as_bf16x8(*reinterpret_cast<const uint4*>(tile + (k / NKS) * 32 * ROWB + row_rd[k % NKS]));
      };
      bf16x8_t ring[PF + 1];
      static_for<0, PF>([&](auto kc) { ring[kc.value] = operand(kc.value); });
      // An E wave runs its matrix steps at raised priority: its path from barrier to barrier is the
      // longer one, and with equal priorities the partner's vector instructions get between its
      // matrix instructions (1.5 % on the kernel; raising the P waves too, or instead: nothing)
      if (!p_wave) __builtin_amdgcn_s_setprio(3);
      static_for<0, 2 * NKS>([&](auto kc) {
        constexpr int k = decltype(kc)::value, ib = k / NKS, ks = k % NKS;
        if constexpr (k + PF < 2 * NKS) ring[(k + PF) % (PF + 1)] = operand(k + PF);
        st2[ib] = E::mfma(ring[k % (PF + 1)], bfrag[ks], st2[ib]);  // the chains start from the exponent offsets (P) or delta (E)
        between(kc);
        __builtin_amdgcn_sched_barrier(0);  // keep the operand reads ahead of their use
      });
      if (!p_wave) __builtin_amdgcn_s_setprio(0);
    };
    // 4 NDB matrix steps of acc += W^T X over the tile's 64 rows (W = pw or ew, X = dO or Q tile).
    // Element e of the A operand is row 16 sl + 8 (e / 4) + 4 hh + e % 4 of its block, so the
    // B operand is the run of four rows starting at 16 sl + 4 hh and the run 8 rows on.
    auto cols_product = [&](const unsigned char* tile, auto&& before) {
      auto operand = [&](int k) {
        const int ib = k / (2 * NDB), sl = (k / NDB) % 2, db = k % NDB;
        const unsigned char* base = tile + (ib * 32 + sl * 16) * ROWB;
        return read_tr_pair(base + tr_lo[db], base + tr_hi[db]);
      };
      bf16x8_t ring[PF + 1];
      static_for<0, PF>([&](auto kc) { ring[kc.value] = operand(kc.value); });
      if (!p_wave) __builtin_amdgcn_s_setprio(3);
      static_for<0, 4 * NDB>([&](auto kc) {
        constexpr int k = decltype(kc)::value, ib = k / (2 * NDB), sl = (k / NDB) % 2, db = k % NDB;
        if constexpr (k + PF < 4 * NDB) ring[(k + PF) % (PF + 1)] = operand(k + PF);
        before(kc);
        const bf16x8_t a = as_bf16x8(make_uint4(w2[ib][4 * sl], w2[ib][4 * sl + 1], w2[ib][4 * sl + 2], w2[ib][4 * sl + 3]));
        acc[db] = E::mfma(a, ring[k % (PF + 1)], acc[db]);
        __builtin_amdgcn_sched_barrier(0);
      });
      if (!p_wave) __builtin_amdgcn_s_setprio(0);
    };

    // dV += P^T dO of tile it - 1 (its dO is still staged: the E waves work on that tile now)
    if (p_wave && it > it_begin) cols_product(Ot, [](auto) {});
    if (p_active) {
      // exponent offsets -LSE log2 e, where the score chains start; masked pairs get -inf: P = 0
      // whatever the score
      floatx16_t (&nl)[2] = st2;
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const float4 L = *reinterpret_cast<const float4*>(&nl_s[ib * 32 + 8 * vq + 4 * hh]);
          constexpr float f = C::OFFSETS ? 1.f : -kLog2e;
          nl[ib][4 * vq + 0] = L.x * f; nl[ib][4 * vq + 1] = L.y * f;
          nl[ib][4 * vq + 2] = L.z * f; nl[ib][4 * vq + 3] = L.w * f;
        }
      // a row whose LSE is -inf saw no key in the whole attention: its offset came out as +inf
      // and must be -inf (P = 0).  One look at the tile's 64 staged values per wave finds the case.
      const bool blind_row = !C::OFFSETS && __builtin_amdgcn_ballot_w64(nl_s[lane] == -INFINITY) != 0;
      if (need_mask || blind_row) {
#pragma unroll
        for (int ib = 0; ib < 2; ++ib)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int i_off = i0 + ib * 32 + acc_row(v, hh);
            if constexpr (C::OFFSETS) {  // (the rows' own reasons are in the offset already, and testing them again took 12 us of 99)
              const bool ok = key_ok && (!isdiag || my_koff <= i_off);
              nl[ib][v] = ok ? nl[ib][v] : -INFINITY;
            } else {
              const bool ok = key_ok && i_off < qlen && (!isdiag || my_koff <= i_off) && nl[ib][v] < INFINITY;
              nl[ib][v] = ok ? nl[ib][v] : -INFINITY;
            }
          }
      }
      auto exps = [&](int ib, int w) {  // elements 2 w, 2 w + 1 of block ib
        const float p0 = fast_exp2(st2[ib][2 * w]);
        const float p1 = fast_exp2(st2[ib][2 * w + 1]);
        w2[ib][w] = E::pack2(p0, p1);
      };
      // S of both blocks; the exponentials of block 0 between the matrix steps of block 1
      rows_product(Qt, [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k >= NKS) static_for<0, 8 / NKS>([&](auto uc) { exps(0, (k - NKS) * (8 / NKS) + uc.value); });
      });
#pragma unroll
      for (int w = 0; w < 8; ++w) exps(1, w);
      // hand P to the partner wave
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
          *reinterpret_cast<uint4*>(xch_w + (ib * 2 + hf) * 1024) =
              make_uint4(w2[ib][4 * hf], w2[ib][4 * hf + 1], w2[ib][4 * hf + 2], w2[ib][4 * hf + 3]);
    } else if (e_active) {
      // T = delta - dO V^T: the chains start from the rows' delta
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const float4 Dl = *reinterpret_cast<const float4*>(&dl_s[ib * 32 + 8 * vq + 4 * hh]);
          st2[ib][4 * vq + 0] = Dl.x; st2[ib][4 * vq + 1] = Dl.y; st2[ib][4 * vq + 2] = Dl.z; st2[ib][4 * vq + 3] = Dl.w;
        }
      rows_product(Ot, [](auto) {});
      uint32_t pw[2][8];
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const uint4 x = *reinterpret_cast<const uint4*>(xch_r + (ib * 2 + hf) * 1024);
          pw[ib][4 * hf] = x.x; pw[ib][4 * hf + 1] = x.y; pw[ib][4 * hf + 2] = x.z; pw[ib][4 * hf + 3] = x.w;
        }
      auto etimes = [&](int ib, int w) {  // E = P o T for elements 2 w, 2 w + 1 of block ib
        w2[ib][w] = E::pack2(E::lo(pw[ib][w]) * st2[ib][2 * w], E::hi(pw[ib][w]) * st2[ib][2 * w + 1]);
      };
#pragma unroll
      for (int w = 0; w < 8; ++w) etimes(0, w);
      // dK += E^T Q; the products of block 1 between the matrix steps of block 0
      cols_product(Qt, [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k < 2 * NDB) static_for<0, 8 / (2 * NDB)>([&](auto uc) { etimes(1, k * (8 / (2 * NDB)) + uc.value); });
      });
    }
    wait_vmcnt<0>();  // this wave's part of the next tile, issued a whole iteration ago
    store_offsets(st_n);
    if (it < it_end) advance(cur);
    const int freed = st_e;
    st_e = st_p; st_p = st_n; st_n = freed;
    const int freed_o = so_e;
    so_e = so_n; so_n = freed_o;
  }

  // ---- several workgroups share this key tile's query loop: all park their partial sums, and the
  // last to arrive adds them up in split order (split_exchange.h)
  if (p.nsplit > 1) {
    int* const role = reinterpret_cast<int*>(smem + C::ROLE_OFF);
    const int tile_id = bhk * p.kt_total + kt;
    constexpr int WAVE_B = NDB * 16 * 64 * 4;  // bytes per wave and part
    unsigned char* parts = reinterpret_cast<unsigned char*>(p.ws_part) + (int64_t)tile_id * p.nsplit * (kBwdWaves * WAVE_B);
    const __amdgpu_buffer_rsrc_t buf = part_buffer(parts);
    const uint32_t mine = wave * WAVE_B + lane * 16;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq)
        store_part(buf, sp * (kBwdWaves * WAVE_B) + mine + (db * 4 + vq) * 1024,
                   floatx4_t{acc[db][4 * vq], acc[db][4 * vq + 1], acc[db][4 * vq + 2], acc[db][4 * vq + 3]});
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) *role = arrive(p.ws_cnt + tile_id, p.nsplit);
    __syncthreads();
    if (*role == kLeaves) return;
    const float start = *role == kGathers ? 0.f : NAN;
    floatx16_t sum[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[db][v] = start;
    for (int s2 = 0; s2 < p.nsplit; ++s2) {
      if (s2 == sp) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) sum[db] += acc[db];
      } else {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const floatx4_t x = load_part(buf, s2 * (kBwdWaves * WAVE_B) + mine + (db * 4 + vq) * 1024);
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[db][4 * vq + r] += x[r];
          }
      }
    }
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = sum[db];
  }

  // ---- dV (P waves) and dK = -scale * (accumulated E^T Q) (E waves) of the wave's 32 keys.
  // A lane owns one column per block and 16 key rows; registers 4 vq .. 4 vq + 3 are four
  // consecutive keys.  Each such group is transposed across the four lanes of a quad (four
  // adjacent columns), so that a lane then holds four adjacent columns of one key and stores
  // 16 bytes: a quarter of the store instructions, which the address unit takes at the same
  // rate whatever their width (stored one float at a time, this epilogue took 3.2 us of a
  // 74 us launch).  This workgroup is the only one that writes these rows in this launch, so
  // accumulation is a plain read-modify-write.
  float* base = (p_wave_s ? tab.step[step].dv : tab.step[step].dk) + (((int64_t)b * p.Hkv + hk) * p.kv_len + kstart) * D;
  const float f = p_wave ? 1.f : -p.scale;
  const bool odd = lane & 1, upper = lane & 2;
  const int col4 = (l32 >> 2) * 4, key_in_group = l32 & 3;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const float r0 = acc[db][4 * vq] * f, r1 = acc[db][4 * vq + 1] * f, r2 = acc[db][4 * vq + 2] * f, r3 = acc[db][4 * vq + 3] * f;
      // lanes one apart exchange (r0, r1) and (r2, r3), then lanes two apart exchange the pairs
      // (every exchange runs in all lanes: a lane reads its partner's register, so none may sit in a branch)
      const float p0 = quad_swap1(r0), p1 = quad_swap1(r1), p2 = quad_swap1(r2), p3 = quad_swap1(r3);
      const float a0 = odd ? p1 : r0, a1 = odd ? r1 : p0, a2 = odd ? p3 : r2, a3 = odd ? r3 : p2;
      const float q0 = quad_swap2(a0), q1 = quad_swap2(a1), q2 = quad_swap2(a2), q3 = quad_swap2(a3);
      float4 x;
      x.x = upper ? q2 : a0; x.y = upper ? q3 : a1; x.z = upper ? a2 : q0; x.w = upper ? a3 : q1;
      const int koff = koff0 + 32 * kg + 8 * vq + 4 * hh + key_in_group;
      if (koff < klen) {
        float4* dst = reinterpret_cast<float4*>(base + (int64_t)koff * D + db * 32 + col4);
        if (p.accumulate) {
          const float4 y = *dst;
          x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
        }
        *dst = x;
      }
    }
}

}  // namespace
}  // namespace loong
