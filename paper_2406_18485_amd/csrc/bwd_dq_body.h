// dQ pass of the backward micro-step on the 16-bit matrix cores (element class E: bf16 or IEEE
// half; the text below says bf16 for both): this step's share of the
// gradient of the local Q chunk, dQ_i += scale * sum_j dS_ij K_j with
// dS_ij = P_ij (dP_ij - delta_i), P recomputed from the final softmax_lse
// (paper: Sec. 3.1 last paragraph; Alg. 2 run backwards).
//
// The workgroups own query rows, exactly like the forward step: eight waves (two per SIMD)
// = NRB row blocks x KS key splits; a wave keeps the Q and dO fragments of its 32 rows and
// the fp32 dQ^T accumulators in registers while K/V tiles stream through LDS (direct
// global -> LDS loads, XOR-permuted 16-byte pieces, NBUF tiles deep).  Per block of 32 keys:
//   S^T  = K Q^T      A = 16-byte LDS reads of K rows,  B = Q fragments
//   dP^T = V dO^T     A = 16-byte LDS reads of V rows,  B = dO fragments
//   dS^T = P^T o (dP^T - delta)   in registers: a lane holds one query row, so the row's
//                     LSE and delta are per-lane scalars; packed to bf16 it is the B operand of
//   dQ^T += K^T dS^T  A = transposing LDS reads of the same K tile.
// Every row belongs to one wave (after the key splits are summed through LDS), so dQ is
// updated with plain loads and stores in a fixed order: the result is reproducible and no
// atomic traffic goes to L2.
#pragma once
#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "loong_internal.h"
#include "row_tiling.h"
#include "split_exchange.h"
#include "step_table.h"
#include "work_map.h"

namespace loong {
namespace {

typedef __attribute__((address_space(3))) void lds_void_t;

struct DqParams {
  const uint16_t *q, *d_o;
  const float *lse, *delta;
  float* dq;
  int B, Hq, Hkv, G, GS;
  int64_t qs[3], ks[3], os[3];
  int q_len;
  Segment qseg[2];
  float scale, c;  // softmax scale; scale * log2(e)
  int overwrite;   // 1: dq is written, not added to
  int ntile[2];    // q tiles per q segment
  int tiles_total;
  int hgroups;     // Hq / GS
  WorkMap map;     // units = batch x head groups, items = q tiles x parts
  int parts;       // workgroups that share the loop over the keys of a q tile
  uint32_t* ws_cnt;  // parts > 1: counter per q tile, zero before and after the launch
  float* ws_part;    // parts > 1: partial dQ of every (q tile, part)
  // both halves in one launch: workgroups of the half that comes first, and whether that is this one
  uint32_t first_grid;
  bool rows_first;
};

// (W: workgroups per unit the form is made for)
template <int D, int KS, int W>
struct DqCfg {
  static constexpr int NRB = kRowWaves / KS;       // 32-row blocks per workgroup
  static constexpr int NJB = KS == 1 ? 2 : 1;      // 32-key blocks per wave and iteration
  static constexpr int BNS = 32 * NJB;             // keys per wave and iteration
  static constexpr int TK = KS * BNS;              // keys staged per iteration
  static constexpr int ROWB = D * 2;               // bytes per K or V row
  static constexpr int CH = D / 8;                 // 16-byte pieces per row
  static constexpr int TILE_B = TK * ROWB;         // bytes of one K (or V) tile
  static constexpr int BUF_B = 2 * TILE_B;
  static constexpr int NBUF = BUF_B * 4 <= 131072 / W ? 4 : 2;
  static constexpr int PD = NBUF - 1;              // tiles in flight ahead of the one being used
  static constexpr int RPI = 1024 / ROWB;          // rows filled by one wave-level load
  static constexpr int KI = TILE_B / 1024 / kRowWaves;  // loads per wave per K (or V) tile
  static constexpr int SLOT_F4 = (D / 32) * 4;     // float4 per lane of one wave's partial result
  static constexpr int TILE_BYTES = NBUF * BUF_B;
  static constexpr int COMB_BYTES = (KS - 1) * NRB * SLOT_F4 * 64 * 16;
  static constexpr int SMEM_BYTES = TILE_BYTES > COMB_BYTES ? TILE_BYTES : COMB_BYTES;
  static_assert(KI >= 1 && KI * 1024 * kRowWaves == TILE_B, "tile must split evenly over the waves");
};

template <class E, int D, int KS, int W>
__device__ __forceinline__ void dq_body(const StepTable& tab, const DqParams& p, uint32_t block, unsigned char* smem) {
  using C = DqCfg<D, KS, W>;
  constexpr int NRB = C::NRB, NJB = C::NJB, BNS = C::BNS, TK = C::TK, NBUF = C::NBUF, PD = C::PD, KI = C::KI;
  constexpr int NDB = D / 32, NKS = D / 16, ROWB = C::ROWB, CH = C::CH;
  // head_dim 64 can run two workgroups per unit (W = 2, four waves per SIMD), in at most 128 registers: the chains' starting values are
  // made by the matrix cores each time (spread) instead of kept in 32 registers, LDS offsets are two registers
  // (row_read_base), one operand is requested ahead, not four, and what only the end needs is found there.  dQ alone, one
  // workgroup per unit -> two: 16384 x 16384 x 8 heads 730 -> 707 us, 1500 x 4100 x 2 x 8 58.8 -> 52.3, 8192 x 8192 x 8
  // 188 -> 195 (256 workgroups); with the offsets added on the vector port instead 728, 57, 205; two operands ahead
  // spilled: 64 us for the second.
  constexpr bool LEAN = W == 2;

  // ---- which (batch, head group, q tile): within a head group the tiles with the most
  // visible keys come first
  int bh, rank;
  if (!decode_work(p.map, block, bh, rank)) return;
  const int tile_rank = rank / p.parts, part = rank - tile_rank * p.parts;
  const int tt = p.tiles_total - 1 - tile_rank;
  const int b = bh / p.hgroups, hg = bh - b * p.hgroups;
  const int qa = tt >= p.ntile[0] ? 1 : 0;
  const int tile = qa ? tt - p.ntile[0] : tt;
  const int BMH = 32 * NRB / p.GS;
  const int row0_wg = tile * BMH;
  const Segment qseg = qa ? p.qseg[1] : p.qseg[0];

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // in a scalar register: what derives from it stays scalar
  const int rb = wave % NRB, ksp = wave / NRB;  // row block, key split
  const int gq = rb % p.GS, rslot = rb / p.GS;
  const int h = hg * p.GS + gq, hk = h / p.G;
  const int wrow0 = row0_wg + rslot * 32;
  const int my_off = wrow0 + l32;
  const bool wave_live = wrow0 < qseg.len;
  const bool row_ok = my_off < qseg.len;
  const int my_row = qseg.start + min(my_off, qseg.len - 1);
  const int last_off_wg = min(row0_wg + BMH, qseg.len) - 1;

  // ---- visible key tiles of this workgroup: the key halves its rows see, one after the other
  const int klen = tab.klen, kend_diag = min(klen, last_off_wg + 1);  // keys of a whole and of the diagonal half
  const uint32_t n_list0 = scalar_now(tab.n_list[0]), n_list1 = scalar_now(tab.n_list[1]);
  const uint32_t n_diag0 = scalar_now(tab.n_diag[0]), n_diag1 = scalar_now(tab.n_diag[1]);
  const uint32_t e00 = scalar_now(tab.first_row[0][0]), e01 = scalar_now(tab.first_row[0][1]);  // the first two entries of either
  const uint32_t e10 = scalar_now(tab.first_row[1][0]), e11 = scalar_now(tab.first_row[1][1]);
  const uint32_t first = qa ? e10 : e00, second = qa ? e11 : e01;
  const int n_list = (int)(qa ? n_list1 : n_list0), n_diag = (int)(qa ? n_diag1 : n_diag0);
  const int all_t = (n_list - n_diag) * ((klen + TK - 1) / TK) + n_diag * ((kend_diag + TK - 1) / TK);
  auto find_dq_row = [&](int off) { return p.dq + b * p.os[0] + h * p.os[1] + (int64_t)(qseg.start + min(off, qseg.len - 1)) * p.os[2]; };
  if (all_t == 0) {  // nothing visible: no share of dQ in this step
    if (p.overwrite && ksp == 0 && row_ok && part == 0) {
      float* const dq_row = find_dq_row(my_off);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
          *reinterpret_cast<float4*>(dq_row + db * 32 + 8 * vq + 4 * hh) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return;
  }

  const int first_t = (int)((int64_t)all_t * part / p.parts), total_t = (int)((int64_t)all_t * (part + 1) / p.parts) - first_t;

  // ---- Q and dO fragments (B operands): row my_row, columns 16 ks + 8 hh .. +7; the row's
  // LSE in log2 units, negated, and its delta.  A row with LSE = -inf sees no key at all.
  bf16x8_t qf[NKS], dof[NKS];
  float nl, dl;
  {
    const int64_t ro = b * p.qs[0] + h * p.qs[1] + (int64_t)my_row * p.qs[2];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      // Q comes with the softmax scale and log2 e folded in (and is rounded to 16 bits again): the
      // score product then ends in the exponent's units and its chain can start from the row's
      // offset (below).  The second rounding moves a recomputed exponent by about 2^-9 of the
      // terms' root sum of squares, a relative change of P well below the 2^-9 that rounding P to
      // 16 bits for the next product costs anyway (the forward pass, whose LSE is compared to
      // 1e-3, keeps the exact multiply-add).
      qf[ks] = scaled_fragment<E>(as_bf16x8(*reinterpret_cast<const uint4*>(p.q + ro + ks * 16 + hh * 8)), p.c);
      dof[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(p.d_o + ro + ks * 16 + hh * 8));
    }
    const int64_t r1 = ((int64_t)b * p.Hq + h) * p.q_len + my_row;
    const float L = p.lse[r1];
    nl = L == -INFINITY ? -INFINITY : L * -kLog2e;
    dl = p.delta[r1];
  }

  floatx16_t ndl;  // -delta of the lane's row in every element: where the dP chains start
  floatx16_t nlt;  // -LSE log2 e of the lane's row in every element: where the score chains start
#pragma unroll
  for (int v = 0; v < 16; ++v) { ndl[v] = -dl; nlt[v] = nl; }  // (LEAN: not used)
  const s16x4_t nl_pieces = pieces_of(nl, lane), ndl_pieces = pieces_of(-dl, lane);
  floatx16_t acc[NDB];  // dQ^T of the wave's rows (without the softmax scale)
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;

  // ---- staging: global -> LDS directly.  Load i of this wave fills LDS bytes
  // [(wave + 8 i) * 1024, +1024) of the K (or V) tile: row (wave + 8 i) * RPI + lane / CH,
  // piece position lane % CH, which holds piece (position ^ swizzle(row)) of that row.
  const int64_t rowbytes = p.ks[2] * 2;
  auto staged_row = [&](int lane) { return wave * C::RPI + lane / CH; };  // inside the tile for i = 0; later loads add 8*RPI rows
  auto staged_piece = [&](int lane) { return (uint32_t)((lane % CH) ^ tile_swizzle<D>(staged_row(lane))) * 16; };
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_t*)smem;  // LDS byte address of the buffers
  // a place in the list of key halves: entry, first key of the tile, end of the half's visible keys
  // (advanced tile by tile: the list is read once per half)
  struct Cursor { uint32_t e; int i, j0, kend; };
  auto enter = [&](Cursor& cu, int i) {
    cu.i = i; cu.j0 = 0;
    cu.e = i ? second : first;
    if (i > 1) cu.e = qa ? tab.row[1][i] : tab.row[0][i];
    cu.kend = cu.e & kDiagEntry ? kend_diag : klen;
  };
  auto advance = [&](Cursor& cu) {  // true: another half begins
    cu.j0 += TK;
    if (cu.j0 < cu.kend || cu.i + 1 >= n_list) return false;
    enter(cu, cu.i + 1);
    return true;
  };
  const uint16_t *const k0 = scalar_now(tab.step[0].k), *const v0 = scalar_now(tab.step[0].v);
  const int64_t head_off = b * p.ks[0] + hk * p.ks[1];
  Cursor ahead, cur;  // the tile to stage next, the tile in use
  const unsigned char *kbase, *vbase;  // first key of the half `ahead` is in
  auto find_bases = [&] {
    const int64_t off = head_off + (int64_t)(entry_half(ahead.e) * klen) * p.ks[2];
    const int step = entry_step(ahead.e);
    const uint16_t *k = k0, *v = v0;
    if (step) { k = scalar_now(tab.step[step].k); v = scalar_now(tab.step[step].v); }
    kbase = reinterpret_cast<const unsigned char*>(k + off);
    vbase = reinterpret_cast<const unsigned char*>(v + off);
  };
  enter(ahead, 0);
  for (int skip = first_t; skip > 0;) {  // (tile first_t exists)
    const int n = (ahead.kend + TK - 1) / TK;
    if (skip < n) ahead.j0 = skip * TK;
    else enter(ahead, ahead.i + 1);
    skip = skip < n ? 0 : skip - n;
  }
  find_bases();
  cur = ahead;
  // byte offsets of this lane's pieces from the first row of a tile (full tiles only; the
  // 32-bit form needs TK rows to span less than 4 GiB, else every tile takes the general path)
  const bool narrow = rowbytes * TK < (int64_t(1) << 32);
  // (LEAN: the first one alone, in one register; else one each: the additions to the bases took 1 % of a step)
  uint32_t ld_off[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i) ld_off[i] = (uint32_t)(staged_row(lane) + (LEAN ? 0 : i * 8 * C::RPI)) * (uint32_t)rowbytes + staged_piece(lane);
  auto issue_tile = [&](int t) {  // stages the tile at `ahead` (the t-th of this workgroup) and moves on
    const int64_t tb = (int64_t)ahead.j0 * rowbytes;
    const int last = klen - 1 - ahead.j0;  // last valid row of the tile (>= 0); later rows repeat it
    const uint32_t kl = smem_base + (t % NBUF) * C::BUF_B + wave * 1024;
    const uint32_t vl = kl + C::TILE_B;
    if (narrow && last >= TK - 1) {  // whole tile: uniform base in scalar registers + per-lane offset
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const int64_t at = tb + (LEAN ? i * 8 * C::RPI * rowbytes : 0);
        load_to_lds_16(kbase + at, ld_off[LEAN ? 0 : i], kl + i * 8192);
        load_to_lds_16(vbase + at, ld_off[LEAN ? 0 : i], vl + i * 8192);
      }
    } else {
      const int ln = LEAN ? lane_again() : lane;
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const int r = min(staged_row(ln) + i * 8 * C::RPI, last);
        const int64_t ro = tb + (int64_t)r * rowbytes + staged_piece(ln);
        load_to_lds_16(kbase + ro, kl + i * 8192);
        load_to_lds_16(vbase + ro, vl + i * 8192);
      }
    }
    if (advance(ahead)) find_bases();
  };

  // ---- LDS read offsets of this lane (bytes inside a tile; the wave's split and the block
  // and slice indices are added as constants: the swizzle repeats every 16 rows)
  // (row operands: row l32 (+32 jb), pieces 2 ks + hh; K^T operands: runs of four keys 4 hh .. 4 hh + 3 and 8 keys on)
  const uint32_t row_rd = row_read_base<D>(lane), tr_rd = tr_read_base<D>(lane);
  uint32_t row_rds[NKS], tr_lo[NDB], tr_hi[NDB];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) row_rds[ks] = row_rd ^ row_read_xor(ks);
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    tr_lo[db] = tr_rd ^ tr_read_xor(db, 0);
    tr_hi[db] = (tr_rd ^ tr_read_xor(db, 1)) + 8 * ROWB;
  }
  if constexpr (!LEAN) {  // (left to itself the compiler forms them anew for every block, on the port that bounds the loop)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm("" : "+v"(row_rds[ks]));
#pragma unroll
    for (int db = 0; db < NDB; ++db) asm("" : "+v"(tr_lo[db]), "+v"(tr_hi[db]));
  }

  // ---- pipeline: PD tiles in flight.  Everything loaded so far is waited for here, so that
  // no counter wait of the compiler's own ends up inside the loop, where it would also wait
  // for the tiles in flight.
  wait_vmcnt<0>();
#pragma unroll
  for (int t = 0; t < PD; ++t)
    if (t < total_t) issue_tile(t);

  for (int t = 0; t < total_t; ++t) {
    // this wave's loads of tile t have landed when at most the later tiles' are outstanding
    const int later = min(PD - 1, total_t - 1 - t);
    if (later >= 2) wait_vmcnt<2 * 2 * KI>();
    else if (later == 1) wait_vmcnt<2 * KI>();
    else wait_vmcnt<0>();
    __syncthreads();  // every wave's part of tile t is in LDS; everyone has finished tile t-1
    if (t + PD < total_t) issue_tile(t + PD);  // into the buffer tile t-1 used

    const int jt = cur.j0;
    const bool isdiag = cur.e & kDiagEntry;
    advance(cur);
    const uint32_t Kt = (t % NBUF) * C::BUF_B + ksp * BNS * ROWB;

#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) {
      // A wave skips a block whose keys lie past the end of the segment or past all of its rows.
      const int j0 = jt + ksp * BNS + jb * 32;
      if (!wave_live || j0 >= klen || (isdiag && j0 > wrow0 + 31)) continue;
      const uint32_t Kb = Kt + jb * 32 * ROWB, row_at = Kb + row_rd, tr_at = Kb + tr_rd;

      // ---- S^T = K Q^T, dP^T = V dO^T (keys x rows: a lane holds one query row).  The K and V
      // row operands are requested PF products ahead (in program order, held there by the
      // scheduling barriers): left to itself the compiler keeps two reads in flight and every
      // pair of products then waits out a full LDS latency.
      floatx16_t s, dp;
      {
        constexpr int NIT = 2 * NKS, PF = LEAN ? 1 : 4;
        auto row_frag = [&](int it) {
          return as_bf16x8(*reinterpret_cast<const uint4*>(smem + (LEAN ? row_at ^ row_read_xor(it >> 1) : Kb + row_rds[it >> 1]) + ((it & 1) ? C::TILE_B : 0)));
        };
        bf16x8_t ring[PF + 1];
        static_for<0, PF>([&](auto i) { ring[i.value] = row_frag(i.value); });
        if constexpr (LEAN) { s = spread(nl_pieces); dp = spread(ndl_pieces); }
        // (the dP chain starts from -delta of the lane's row, so it ends as dP - delta; the score
        // chain from -LSE log2 e, so it ends as the exponent of P: two vector instructions per
        // element that the matrix cores do on the side)
        static_for<0, NIT>([&](auto i) {
          constexpr int it = i.value, ks = it >> 1;
          if constexpr (it + PF < NIT) ring[(it + PF) % (PF + 1)] = row_frag(it + PF);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (it & 1) dp = E::mfma(ring[it % (PF + 1)], dof[ks], ks || LEAN ? dp : ndl);
          else s = E::mfma(ring[it % (PF + 1)], qf[ks], ks || LEAN ? s : nlt);
        });
      }
      // ---- dS^T = P^T (dP^T - delta), the softmax scale is applied to the sums at the end
      float e[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) e[v] = fast_exp2(s[v]) * dp[v];
      if (j0 + 32 > klen || (isdiag && j0 + 31 > wrow0)) {  // diagonal or ragged end only
        const int ln = LEAN ? lane_again() : lane, off = wrow0 + (ln & 31);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = j0 + acc_row(v, ln >> 5);
          const bool ok = key < klen && (!isdiag || key <= off);
          e[v] = ok ? e[v] : 0.f;
        }
      }
      uint4 pk[2];
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
        pk[sl] = make_uint4(E::pack2(e[8 * sl + 0], e[8 * sl + 1]), E::pack2(e[8 * sl + 2], e[8 * sl + 3]),
                            E::pack2(e[8 * sl + 4], e[8 * sl + 5]), E::pack2(e[8 * sl + 6], e[8 * sl + 7]));
      // ---- dQ^T += K^T dS^T.  Element e of the B operand is key 16 sl + 8 (e / 4) + 4 hh + e % 4
      // of the block: the A operand is the run starting at key 16 sl + 4 hh and the run 8 keys on.
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const unsigned char* kp = smem + sl * 16 * ROWB;
          const bf16x8_t k_cols = LEAN ? read_tr_pair(kp + (tr_at ^ tr_read_xor(db, 0)), kp + 8 * ROWB + (tr_at ^ tr_read_xor(db, 1)))
                                       : read_tr_pair(kp + Kb + tr_lo[db], kp + Kb + tr_hi[db]);
          acc[db] = E::mfma(k_cols, as_bf16x8(pk[sl]), acc[db]);
        }
    }
  }

  // ---- sum the key splits: splits 1.. park their dQ^T in LDS, split 0 adds them in order.
  // Split 0 requests its rows of dQ first: the round trip to memory runs while the others park.
  // (the lane's place is found anew: at head_dim 64 the loop has no register to spare for it)
  const int end_lane = lane_again(), end_off = wrow0 + (end_lane & 31), end_hh = end_lane >> 5;
  const bool end_ok = end_off < qseg.len;
  float* const dq_row = find_dq_row(end_off);
  float4 old[NDB][4];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) old[db][vq] = make_float4(0.f, 0.f, 0.f, 0.f);
  // (One branch around all the loads: with one around each, they are waited for one by one, 8192 rows x 100 keys
  // x 8 heads without a split 31.9 us instead of 24.6.)
  auto request_old = [&] {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) old[db][vq] = *reinterpret_cast<const float4*>(dq_row + db * 32 + 8 * vq + 4 * end_hh);
  };
  if (ksp == 0 && end_ok && !p.overwrite && p.parts == 1) request_old();
  if (KS > 1) {
    __syncthreads();  // all reads of the last tile are done: the tile buffers are reused
    float4* slots = reinterpret_cast<float4*>(smem);
    if (ksp > 0) {
      float4* mine = slots + ((ksp - 1) * NRB + rb) * C::SLOT_F4 * 64 + end_lane;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
          mine[(db * 4 + vq) * 64] = make_float4(acc[db][4 * vq], acc[db][4 * vq + 1], acc[db][4 * vq + 2], acc[db][4 * vq + 3]);
    }
    __syncthreads();
    if (ksp > 0 && p.parts == 1) return;
#pragma unroll 1
    for (int sp = 1; sp < KS && ksp == 0; ++sp) {
      const float4* theirs = slots + ((sp - 1) * NRB + rb) * C::SLOT_F4 * 64 + end_lane;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const float4 x = theirs[(db * 4 + vq) * 64];
          acc[db][4 * vq + 0] += x.x; acc[db][4 * vq + 1] += x.y;
          acc[db][4 * vq + 2] += x.z; acc[db][4 * vq + 3] += x.w;
        }
    }
  }

  // ---- several workgroups share the keys of this tile: all park their sums, and the last to arrive adds them up in order
  // (split_exchange.h)
  if (p.parts > 1) {
    int* const role = reinterpret_cast<int*>(smem + C::TILE_BYTES - 16);
    static_assert(C::COMB_BYTES <= C::TILE_BYTES - 16, "nobody reads there any more");
    constexpr int WAVE_B = NDB * 16 * 64 * 4;  // bytes per row block and part
    const int tile_id = bh * p.tiles_total + tt;
    const __amdgpu_buffer_rsrc_t buf = part_buffer(reinterpret_cast<unsigned char*>(p.ws_part) + (int64_t)tile_id * p.parts * (NRB * WAVE_B));
    const uint32_t mine = rb * WAVE_B + end_lane * 16;
    if (ksp == 0) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
          store_part(buf, part * (NRB * WAVE_B) + mine + (db * 4 + vq) * 1024,
                     floatx4_t{acc[db][4 * vq], acc[db][4 * vq + 1], acc[db][4 * vq + 2], acc[db][4 * vq + 3]});
    }
    wait_vmcnt<0>();
    __syncthreads();
    if (wave == 0 && end_lane == 0) *role = arrive(p.ws_cnt + tile_id, p.parts);
    __syncthreads();
    if (ksp > 0 || *role == kLeaves) return;
    const float start = *role == kGathers ? 0.f : NAN;
    // (32 columns at a time, of NDB parts in flight, the own one among them: the sums of all columns beside the own ones made every
    // dQ kernel keep 9 registers in scratch memory)
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      floatx16_t sum;
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[v] = start;
#pragma unroll 1
      for (int s2 = 0; s2 < p.parts; s2 += NDB) {
        floatx4_t x[NDB][4];
#pragma unroll
        for (int u = 0; u < NDB; ++u)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) x[u][vq] = load_part(buf, min(s2 + u, p.parts - 1) * (NRB * WAVE_B) + mine + (db * 4 + vq) * 1024);
#pragma unroll
        for (int u = 0; u < NDB; ++u)
          if (s2 + u < p.parts) {
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] += x[u][v >> 2][v & 3];
          }
      }
      acc[db] = sum;
    }
    if (end_ok && !p.overwrite) request_old();
  }

  // ---- dQ row += scale * sum: register 4 vq + r of block db is column 32 db + 8 vq + 4 hh + r
  if (end_ok) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        float4* dst = reinterpret_cast<float4*>(dq_row + db * 32 + 8 * vq + 4 * end_hh);
        float4 x = old[db][vq];
        x.x = fmaf(acc[db][4 * vq + 0], p.scale, x.x); x.y = fmaf(acc[db][4 * vq + 1], p.scale, x.y);
        x.z = fmaf(acc[db][4 * vq + 2], p.scale, x.z); x.w = fmaf(acc[db][4 * vq + 3], p.scale, x.w);
        *dst = x;
      }
  }
}

}  // namespace
}  // namespace loong
