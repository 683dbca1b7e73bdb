"""Single-GPU replay of one device's share of Double-Ring-Attention.

The ring is simulated by visiting the K/V chunks, all resident in HBM, in the order in
which the inner and outer rings of Alg. 2 would deliver them to the simulated rank.  The
forward takes runs of visits per launch, one after the other, with the bits of a launch per visit; the
backward, whose visits only share sums, runs of visits in no order, since every chunk is there.  torch is used
for device memory and the stream only.
"""
from __future__ import annotations

from dataclasses import dataclass

import torch

from . import binding as B


@dataclass
class RingShape:
    cp: int
    w: int
    rank: int
    hq: int
    hkv: int
    d: int
    c: int
    dtype: int          # B.BF16 | B.FP32 | B.FP16
    scale: float
    batch: int = 1
    extra_flags: int = 0   # OR-ed into every step descriptor (e.g. binding.key_splits(n))

    @property
    def L(self) -> int:
        return 2 * self.c


def visit_plan(shape: RingShape) -> list[dict]:
    """Per micro-step: source rank, chunk ids and block classes, from the library."""
    return [B.zigzag_mask(shape.cp, shape.w, shape.rank, t) for t in range(shape.cp)]


def _desc(shape: RingShape, step: dict, flags: int) -> B.StepDesc:
    return B.make_desc(batch=shape.batch, n_q_heads=shape.hq, n_kv_heads=shape.hkv, head_dim=shape.d,
                       q_len=shape.L, kv_len=shape.L, dtype=shape.dtype, softmax_scale=shape.scale,
                       causal=True, chunk_len=shape.c, q_chunk=step["q_chunk"], kv_chunk=step["kv_chunk"],
                       flags=flags | shape.extra_flags)


def _visited(chunks, order, last):
    """chunks[src] for every src of `order` (the largest is `last`), of a stacked tensor their device pointers (it is not sliced for it).  The
    items themselves are returned, not their pointers: one that `chunks` made for this call lives until it has been used."""
    if isinstance(chunks, torch.Tensor):
        if last >= chunks.shape[0]:
            raise IndexError(f"source rank {last} is out of range of {chunks.shape[0]} chunks")
        base, step = chunks.data_ptr(), chunks.stride(0) * chunks.element_size()
        return B.pointer_array([base + src * step for src in order])
    return [chunks[src] for src in order]


class RingReplay:
    """Buffers and launch sequence of the forward and backward replay for one rank.

    k_by_src / v_by_src: [cp, batch, hkv, L, d] device tensors holding, for every source
    rank, its zigzag chunk pair (low half first).  q, d_o: [batch, hq, L, d].
    """

    def __init__(self, shape: RingShape, device="cuda:0"):
        self.shape = shape
        self.dev = torch.device(device)
        self.plan = visit_plan(shape)
        s = shape
        f32 = dict(dtype=torch.float32, device=self.dev)
        self.store_dtype = {B.BF16: torch.bfloat16, B.FP16: torch.float16, B.FP32: torch.float32}[s.dtype]
        self.rows = s.batch * s.hq * s.L
        self.out = torch.empty(s.batch, s.hq, s.L, s.d, **f32)      # running fp32 output
        self.lse = torch.empty(s.batch, s.hq, s.L, **f32)
        self.o = torch.empty(s.batch, s.hq, s.L, s.d, dtype=self.store_dtype, device=self.dev)
        self.delta = torch.empty(s.batch, s.hq, s.L, **f32)
        self.dq = torch.empty(s.batch, s.hq, s.L, s.d, **f32)
        self.dk = torch.empty(s.cp, s.batch, s.hkv, s.L, s.d, **f32)  # per source rank
        self.dv = torch.empty(s.cp, s.batch, s.hkv, s.L, s.d, **f32)
        self.block_out = None
        self.block_lse = None
        self.workspace, self._workspaces = None, []   # (one that was outgrown may be in use on some stream: it is kept)
        self._prepare()

    # ---- what the calls take of the shape and the plan, kept between them
    def _prepare(self):
        s = self.shape
        self._prepared = dict(vars(s)), [dict(step) for step in self.plan]
        self._order = [step["src_rank"] for step in self.plan]
        self._last, self._repeats = max(self._order), len(set(self._order)) < len(self._order)
        descs = B.StepDesc * len(self.plan)
        self._fwd_descs = descs(*(_desc(s, step, 0) for step in self.plan))
        # the same where every step is a call: the first writes the running result, the others merge into it
        self._merge_descs = descs.from_buffer_copy(self._fwd_descs)
        for desc in self._merge_descs[1:]:
            desc.flags |= B.FUSE_MERGE
        # the backward steps of a pass: the first forms delta and writes dq, and all are one run
        self._bwd_descs = descs.from_buffer_copy(self._fwd_descs)
        for desc in self._bwd_descs:
            desc.flags |= B.COMPUTE_DELTA | B.OVERWRITE_DQ
        # caller-owned scratch of the backward steps: the largest any micro-step, or all in one run, ask for
        need = max(B.workspace_bytes_steps(self._bwd_descs), *(B.workspace_bytes(desc) for desc in self._fwd_descs))
        if self.workspace is not None and self.workspace.numel() >= need:
            return
        # (nothing is cleared here: every call clears its counters on its own stream, and a clearing on this one could come
        # while a call on another counts.  Where no step needs any: 16 bytes that none of them touches.)
        self._workspaces.append(torch.empty(need, dtype=torch.uint8, device=self.dev) if need else
                                torch.zeros(16, dtype=torch.uint8, device=self.dev))
        self.workspace = self._workspaces[-1]

    def _follow(self):
        """The program may have changed `shape` (its scale, its extra flags) or `plan` since the last call."""
        if vars(self.shape) != self._prepared[0] or self.plan != self._prepared[1]:
            self._prepare()

    # ---- forward: cp x (Attention [+ Update]) then the cast to the stored activation type
    def forward(self, q, k_by_src, v_by_src, fuse_merge=True, stream=None):
        s = self.shape
        self._follow()
        if fuse_merge:
            # the first visit writes the running result (rows that see nothing get the neutral
            # element), the later ones merge into it (no separate initialisation), the last stores o too
            k, v = (_visited(x, self._order, self._last) for x in (k_by_src, v_by_src))
            B.attn_steps_fwd(self._fwd_descs, q, k, v, self.out, self.lse, self.o, stream)
            return
        if self.block_out is None:
            self.block_out = torch.empty_like(self.out)
            self.block_lse = torch.empty_like(self.lse)
        # the first step writes the running result (an update of the neutral element would give its very bits), the
        # others are merged into it: two launches fewer, 11 us of 97 in 3 steps of 12 heads x 1554 rows
        for t, (desc, src) in enumerate(zip(self._fwd_descs, self._order)):
            out, lse = (self.block_out, self.block_lse) if t else (self.out, self.lse)
            B.attn_step_fwd(desc, q, k_by_src[src], v_by_src[src], out, lse, stream)
            if t:
                B.lse_merge(self.rows, s.d, self.out, self.lse, out, lse, stream)
        B.finalize_out(self.rows, s.d, self.out, self.o, s.dtype, stream)

    # ---- backward from the stored O and LSE: delta once, then the cp steps, whose chunks are all here, as one run
    def backward(self, q, k_by_src, v_by_src, d_o, stream=None):
        self._follow()
        if self.shape.extra_flags & B.BWD_ONLY_DKV:   # (the steps leave dq alone)
            self.dq.zero_()
        k, v, dk, dv = (_visited(x, self._order, self._last) for x in (k_by_src, v_by_src, self.dk, self.dv))
        if self._repeats:   # the steps of a run need gradients of their own: one after the other
            for t, desc in enumerate(self._bwd_descs):
                step = B.StepDesc.from_buffer_copy(desc)
                if t:
                    step.flags &= ~(B.COMPUTE_DELTA | B.OVERWRITE_DQ)
                B.attn_step_bwd(step, q, k[t], v[t], self.o, d_o, self.lse, self.delta, self.dq, dk[t], dv[t], self.workspace,
                                stream=stream)
            return
        B.attn_steps_bwd(self._bwd_descs, q, k, v, self.o, d_o, self.lse, self.delta, self.dq, dk, dv, self.workspace,
                         stream=stream)

    # ---- forward with the receive buffers of Alg. 2: the chunk of the next micro-step arrives
    # in an inner-ring buffer while the current one is used, and the first chunk of the next
    # outer step arrives in the outer-ring buffer during the whole inner ring.  On one GPU the
    # "transfers" are device-to-device copies from the resident chunks on two side streams
    # (default priority), ordered against the step kernels with events exactly as the P2P
    # receives would be.  Result: the same (out, lse, o) as forward().
    def forward_two_buffers(self, q, k_by_src, v_by_src):
        s = self.shape
        main = torch.cuda.current_stream(self.dev)
        if not hasattr(self, "_kv_bufs"):
            shp = (s.batch, s.hkv, s.L, s.d)
            self._kv_bufs = [(torch.empty(shp, dtype=self.store_dtype, device=self.dev),
                              torch.empty(shp, dtype=self.store_dtype, device=self.dev)) for _ in range(3)]
            self._comm = (torch.cuda.Stream(self.dev), torch.cuda.Stream(self.dev))   # inner ring, outer ring
            self._events = [torch.cuda.Event() for _ in range(3)], [torch.cuda.Event() for _ in range(3)]
        self._follow()
        bufs, (inner, outer), (filled, released) = self._kv_bufs, self._comm, self._events

        # (this path is bound by the host where chunks are short, and a stream context costs 8 us: more than the step's launch)
        def receive(stream, b, src):
            stream.wait_event(released[b])          # the buffer's last reader has finished
            torch.cuda.set_stream(stream)
            try:
                bufs[b][0].copy_(k_by_src[src], non_blocking=True)
                bufs[b][1].copy_(v_by_src[src], non_blocking=True)
            finally:
                torch.cuda.set_stream(main)
            filled[b].record(stream)

        for ev in released:
            ev.record(main)
        cur, nxt, out = 0, 1, 2
        receive(inner, cur, self.plan[0]["src_rank"])   # the own chunk
        n_outer = s.cp // s.w
        for t in range(len(self.plan)):
            a, b = divmod(t, s.w)
            if b == 0 and a + 1 < n_outer:
                receive(outer, out, self.plan[(a + 1) * s.w]["src_rank"])
            if b + 1 < s.w:
                receive(inner, nxt, self.plan[t + 1]["src_rank"])
            main.wait_event(filled[cur])
            if t + 1 < len(self.plan):
                B.attn_step_fwd(self._merge_descs[t], q, bufs[cur][0], bufs[cur][1], self.out, self.lse)
            else:   # the last one stores o too
                last = (B.StepDesc * 1)(self._merge_descs[t])
                B.attn_steps_fwd(last, q, bufs[cur][:1], bufs[cur][1:], self.out, self.lse, self.o)
            released[cur].record(main)
            if b + 1 < s.w:
                cur, nxt = nxt, cur
            else:
                cur, out = out, cur
