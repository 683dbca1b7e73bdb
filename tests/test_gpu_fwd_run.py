"""A run of forward micro-steps (attn_steps_fwd) against the same steps one by one and the cast of the result: the
same kernels in the same order, so out, lse and o must be equal bit for bit.  Ranks whose last step leaves
rows without keys, ragged tiles, each forced key split, head groups, a run that continues an earlier one."""
import pytest
import torch

import paper_2406_18485_amd as P
from gpu_harness import DEV, token_major
from paper_2406_18485_amd.ring import RingReplay, RingShape, _desc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,code", [(torch.bfloat16, P.BF16), (torch.float16, P.FP16), (torch.float32, P.FP32)])
@pytest.mark.parametrize("cp,w,rank,hq,hkv,d,c,batch,ks", [
    (4, 2, 0, 4, 1, 128, 200, 1, 0), (4, 4, 3, 2, 2, 64, 33, 2, 4), (3, 3, 1, 6, 2, 128, 129, 1, 2), (2, 1, 1, 8, 8, 64, 1, 1, 1),
    (1, 1, 0, 4, 2, 128, 65, 1, 0), (2, 2, 0, 2, 1, 64, 300, 3, 1)])
def test_run_equals_its_steps_and_the_cast(cp, w, rank, hq, hkv, d, c, batch, ks, dtype, code):
    rep = RingReplay(RingShape(cp=cp, w=w, rank=rank, hq=hq, hkv=hkv, d=d, c=c, dtype=code, scale=d ** -0.5, batch=batch,
                               extra_flags=P.key_splits(ks)), DEV)
    g = torch.Generator(device=DEV).manual_seed(c)
    mk = lambda *s: torch.randn(*s, device=DEV, generator=g).to(dtype)
    q, k, v = mk(batch, hq, 2 * c, d), mk(cp, batch, hkv, 2 * c, d), mk(cp, batch, hkv, 2 * c, d)
    for t in (rep.out, rep.lse, rep.o):
        t.fill_(5.0)
    rep.forward(q, k, v)
    got = [t.clone() for t in (rep.out, rep.lse, rep.o)]

    def step_by_step(first):
        for t, step in enumerate(rep.plan):
            src = step["src_rank"]
            P.attn_step_fwd(_desc(rep.shape, step, P.FUSE_MERGE if first or t else 0), q, k[src], v[src], rep.out, rep.lse)
        P.finalize_out(rep.rows, d, rep.out, rep.o, code)

    step_by_step(0)
    assert all(torch.equal(a, b) for a, b in zip(got, (rep.out, rep.lse, rep.o)))
    # continuing from that result: the first step merges too
    start = [t.clone() for t in (rep.out, rep.lse)]
    step_by_step(1)
    want = [t.clone() for t in (rep.out, rep.lse, rep.o)]
    rep.out.copy_(start[0]); rep.lse.copy_(start[1])
    order = [s["src_rank"] for s in rep.plan]
    descs = (P.StepDesc * cp)(*(_desc(rep.shape, s, P.FUSE_MERGE) for s in rep.plan))
    P.attn_steps_fwd(descs, q, [k[s] for s in order], [v[s] for s in order], rep.out, rep.lse, rep.o)
    assert all(torch.equal(a, b) for a, b in zip(want, (rep.out, rep.lse, rep.o)))


@pytest.mark.parametrize("code,dtype", [(P.BF16, torch.bfloat16), (P.FP16, torch.float16), (P.FP32, torch.float32)])
@pytest.mark.parametrize("cp,w,rank,hq,hkv,d,c,batch,ks", [
    (33, 33, 20, 2, 1, 64, 5, 1, 0), (40, 8, 39, 4, 1, 128, 3, 1, 0),   # more steps than one launch takes
    (5, 5, 2, 4, 2, 128, 257, 2, 1), (5, 5, 2, 4, 2, 128, 257, 2, 2), (6, 3, 4, 3, 1, 64, 97, 1, 2), (6, 2, 0, 3, 3, 64, 130, 1, 1),
    (3, 3, 1, 8, 8, 128, 2048, 1, 0)])   # diagonal step with four splits, one with two, one with four: three launches
def test_runs_over_several_launches_equal_their_steps(cp, w, rank, hq, hkv, d, c, batch, ks, code, dtype):
    """Steps that share a launch hand the running result on in registers, between launches it goes through memory: the same bits."""
    test_run_equals_its_steps_and_the_cast(cp, w, rank, hq, hkv, d, c, batch, ks, dtype, code)


@pytest.mark.parametrize("dtype,code", [(torch.bfloat16, P.BF16), (torch.float16, P.FP16)])
@pytest.mark.parametrize("cp,rank,hq,c,batch", [(3, 0, 8, 1793, 1), (2, 1, 4, 1153, 4), (1, 0, 8, 1152, 1), (2, 0, 8, 1151, 1)])
def test_lines_asked_for_ahead_change_nothing(cp, rank, hq, c, batch, dtype, code):
    """Every head with keys of its own, chunks either side of 2304 keys, a full chip: some lines are requested early, by
    workgroups of a full and a ragged tile.  A forced split of four takes the same path, so the comparison is with groups of one head
    each, which leave the chip too empty for it: the same bits."""
    shape = dict(cp=cp, w=cp, rank=rank, d=128, c=c, dtype=code, scale=128 ** -0.5, extra_flags=P.key_splits(4))
    g = torch.Generator(device=DEV).manual_seed(c)
    mk = lambda *s: torch.randn(*s, device=DEV, generator=g).to(dtype)
    q, k, v = mk(batch, hq, 2 * c, 128), mk(cp, batch, hq, 2 * c, 128), mk(cp, batch, hq, 2 * c, 128)
    rep = RingReplay(RingShape(hq=hq, hkv=hq, batch=batch, **shape), DEV)
    rep.forward(q, k, v)
    for b in range(batch):
        for h in range(hq):
            one = RingReplay(RingShape(hq=1, hkv=1, batch=1, **shape), DEV)
            one.forward(q[b:b + 1, h:h + 1].contiguous(), k[:, b:b + 1, h:h + 1].contiguous(), v[:, b:b + 1, h:h + 1].contiguous())
            assert torch.equal(one.out[0, 0], rep.out[b, h]) and torch.equal(one.lse[0, 0], rep.lse[b, h]) and torch.equal(one.o[0, 0], rep.o[b, h])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lq,hq,hkv", [(2048, 8, 8), (2049, 8, 8), (2304, 8, 2), (4500, 6, 2), (9000, 8, 8)])
def test_a_step_of_any_number_of_rounds_takes_one_of_the_key_splits(lq, hq, hkv, d):
    """Row counts either side of one, two and more rounds of workgroups: the split chosen for them must be one of the
    three forms (bit for bit), and those agree to what rounding P to 16 bits relative to other maxima leaves."""
    lk = 333
    g = torch.Generator(device=DEV).manual_seed(lq + d)
    mk = lambda *s: (torch.randn(*s, device=DEV, generator=g) * 0.5).to(torch.bfloat16)
    q, k, v = mk(1, hq, lq, d), mk(1, hkv, lk, d), mk(1, hkv, lk, d)
    res = []
    for ks in (0, 1, 2, 4):
        out, lse = torch.full((1, hq, lq, d), 3.0, device=DEV), torch.empty(1, hq, lq, device=DEV)
        P.attn_step_fwd(P.make_desc(batch=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, q_len=lq, kv_len=lk, dtype=P.BF16,
                                    softmax_scale=d ** -0.5, flags=P.key_splits(ks)), q, k, v, out, lse)
        res.append((out, lse))
    assert any(torch.equal(res[0][0], o) and torch.equal(res[0][1], l) for o, l in res[1:])
    for o, l in res[1:]:
        assert float((o - res[0][0]).abs().max()) < 4e-3 and float((l - res[0][1]).abs().max()) < 1e-5


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lq,hq,hkv,ks", [(2048, 8, 8, 4), (2304, 8, 8, 4), (3000, 8, 2, 4), (4500, 8, 8, 2), (9000, 8, 8, 1)])
def test_the_split_is_the_smallest_that_fills_the_chip(lq, hq, hkv, ks, d):
    """The key split decides the result's last bits: it is the smallest that puts a workgroup of 32 * 8 / ks rows on at least 7/8
    of 256 units, here 32 * 8 = 256, 288, 376, 288 and 288 workgroups (72 to 192 with the next smaller one)."""
    g = torch.Generator(device=DEV).manual_seed(lq + d)
    mk = lambda *s: (torch.randn(*s, device=DEV, generator=g) * 0.5).to(torch.bfloat16)
    q, k, v = mk(1, hq, lq, d), mk(1, hkv, 700, d), mk(1, hkv, 700, d)
    res = []
    for forced in (0, ks):
        out, lse = torch.empty(1, hq, lq, d, device=DEV), torch.empty(1, hq, lq, device=DEV)
        P.attn_step_fwd(P.make_desc(batch=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, q_len=lq, kv_len=700, dtype=P.BF16,
                                    softmax_scale=d ** -0.5, flags=P.key_splits(forced)), q, k, v, out, lse)
        res.append((out, lse))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("dtype,code", [(torch.bfloat16, P.BF16), (torch.float16, P.FP16)])
@pytest.mark.parametrize("cp,rank,hq,hkv,d,c,batch,ks", [(4, 2, 4, 1, 128, 200, 1, 0), (2, 0, 2, 2, 64, 33, 2, 4), (3, 1, 6, 2, 128, 129, 1, 2), (2, 1, 8, 8, 64, 97, 1, 1)])
def test_strided_tensors_on_another_stream_give_the_same_bits(cp, rank, hq, hkv, d, c, batch, ks, dtype, code):
    """Token-major q, k, v and `out` with gaps between the rows, and the contiguous `o` that the last step stores beside them."""
    shape = RingShape(cp=cp, w=cp, rank=rank, hq=hq, hkv=hkv, d=d, c=c, dtype=code, scale=d ** -0.5, batch=batch, extra_flags=P.key_splits(ks))
    rep = RingReplay(shape, DEV)
    g = torch.Generator(device=DEV).manual_seed(c)
    mk = lambda h: torch.randn(batch, h, 2 * c, d, device=DEV, generator=g).to(dtype)
    q, k, v = mk(hq), [mk(hkv) for _ in range(cp)], [mk(hkv) for _ in range(cp)]
    rep.forward(q, k, v)
    qs, q_stride = token_major(q, 8)
    ks_, vs_ = ([token_major(x, 16)[0] for x in y] for y in (k, v))
    out, o_stride = token_major(torch.full_like(rep.out, 5.0), 4)
    lse, o = torch.full_like(rep.lse, 5.0), torch.full_like(rep.o, 5.0)
    descs = (P.StepDesc * cp)(*(_desc(shape, step, 0) for step in rep.plan))
    for desc in descs:
        desc.q_stride[:], desc.kv_stride[:], desc.o_stride[:] = q_stride, ks_[0].stride()[:3], o_stride
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    order = [s["src_rank"] for s in rep.plan]
    P.attn_steps_fwd(descs, qs, [ks_[s] for s in order], [vs_[s] for s in order], out, lse, o, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(out, rep.out) and torch.equal(lse, rep.lse) and torch.equal(o, rep.o)
    gaps = out.permute(0, 2, 1, 3).as_strided((batch, 2 * c, hq, 4), (out.stride(0), out.stride(2), out.stride(1), 1), d)
    assert bool(gaps.isnan().all())


@pytest.mark.parametrize("lq", [1, 64, 2048, 2049])
@pytest.mark.parametrize("lk", [1, 127, 128, 129, 300, 513, 1000])
def test_either_depth_of_staged_tiles_gives_the_same_bits(lq, lk):
    """head_dim 64 with four key splits: tiles four deep in up to 256 workgroups of 64 rows, two deep in more.  The head of a launch
    of the first kind equals the same head in one of the second, key counts either side of one to four tiles of 128."""
    g = torch.Generator(device=DEV).manual_seed(lq + lk)
    mk = lambda n: (torch.randn(1, n, 64, device=DEV, generator=g) * 0.5).to(torch.bfloat16)
    q, k, v = mk(lq), mk(lk), mk(lk)
    res = []
    for batch in (1, -(-257 // (-(-lq // 64)))):   # `batch` copies of the first head are more than 256 workgroups
        rep = lambda x: x[:1].expand(batch, -1, -1)[:, None].contiguous()
        out, lse = torch.empty(batch, 1, lq, 64, device=DEV), torch.empty(batch, 1, lq, device=DEV)
        P.attn_step_fwd(P.make_desc(batch=batch, n_q_heads=1, n_kv_heads=1, head_dim=64, q_len=lq, kv_len=lk, dtype=P.BF16,
                                    softmax_scale=0.125, flags=P.key_splits(4)), rep(q), rep(k), rep(v), out, lse)
        res.append((out[0], lse[0], out[-1], lse[-1]))
    assert all(torch.equal(a, b) for a, b in zip(*res))
    s = (q[0].double() @ k[0].double().t().contiguous()) * 0.125
    assert float((res[0][0][0] - torch.softmax(s, -1) @ v[0].double()).abs().max()) < 2e-2
