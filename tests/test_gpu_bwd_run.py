"""A run of backward micro-steps in one launch (attn_steps_bwd) against the same steps one by one: rows whose
loop crosses chunk ends of every remainder, key halves nobody sees, shared query loops, more steps than one
launch takes, dq and dk/dv added to, no mask, each forced key split.

Both compute the same sums of the same products (probabilities rounded to 16 bits alike); only the order of
fp32 additions differs (dq over steps in registers, dk/dv in other splits).  An element is a chain of one addition per 16
products (4 in fp32 storage, dealt over four or eight waves): at most 640 here (8 steps x 1280 keys), each rounded by at
most 2^-24 of the running sum, so two orders differ by at most 2 * 640 * 2^-24 = 7.6e-5 of the largest running sum, which
is about the largest element; the result is compared to 1e-4 of that."""
import ctypes as C

import pytest
import torch

import paper_2406_18485_amd as P
from gpu_harness import DEV, token_major
from paper_2406_18485_amd.ring import RingReplay, RingShape, _desc

pytestmark = pytest.mark.gpu


def _close(a, b, tol=1e-4):
    assert torch.isfinite(a).all()
    assert float((a - b).abs().max()) <= tol * float(b.abs().max())


def _replay(cp, w, rank, hq, hkv, d, c, batch, flags=0, dtype=torch.bfloat16, code=P.BF16):
    rep = RingReplay(RingShape(cp=cp, w=w, rank=rank, hq=hq, hkv=hkv, d=d, c=c, dtype=code, scale=d ** -0.5, batch=batch,
                               extra_flags=flags), DEV)
    g = torch.Generator(device=DEV).manual_seed(cp * 1000 + c)
    mk = lambda *s: (torch.randn(*s, device=DEV, generator=g) * 0.5).to(dtype)
    q, d_o = mk(batch, hq, 2 * c, d), mk(batch, hq, 2 * c, d)
    k, v = mk(cp, batch, hkv, 2 * c, d), mk(cp, batch, hkv, 2 * c, d)
    rep.forward(q, k, v)
    return rep, q, k, v, d_o


@pytest.mark.parametrize("cp,w,rank,hq,hkv,d,c,batch,ks", [
    (4, 2, 2, 4, 1, 128, 200, 1, 0), (4, 4, 0, 2, 2, 64, 33, 2, 0), (3, 3, 2, 6, 2, 64, 129, 1, 0), (2, 1, 1, 8, 8, 128, 1, 1, 0),
    (8, 4, 7, 3, 1, 128, 65, 1, 1), (8, 8, 4, 4, 2, 64, 127, 1, 2), (5, 5, 3, 8, 1, 128, 96, 1, 4), (40, 8, 11, 2, 1, 64, 40, 1, 0),
    (8, 8, 3, 8, 8, 128, 640, 1, 0), (6, 3, 5, 8, 4, 64, 512, 3, 0), (1, 1, 0, 4, 2, 128, 300, 1, 0)])
def test_run_equals_its_steps(cp, w, rank, hq, hkv, d, c, batch, ks):
    rep, q, k, v, d_o = _replay(cp, w, rank, hq, hkv, d, c, batch, P.key_splits(ks))
    for t in (rep.dq, rep.dk, rep.dv):
        t.fill_(9.0)
    rep.backward(q, k, v, d_o)
    got = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    if P.workspace_bytes_steps(rep._bwd_descs) > 0:   # (else the run does not count, and leaves the memory alone)
        assert int(rep.workspace[:P.binding.WORKSPACE_HEAD].max()) == 0   # counters are left clean
    rep.backward(q, k, v, d_o)
    assert all(torch.equal(a, b) for a, b in zip(got, (rep.dq, rep.dk, rep.dv)))
    for t, step in enumerate(rep.plan):
        src = step["src_rank"]
        P.attn_step_bwd(_desc(rep.shape, step, 0 if t else P.OVERWRITE_DQ), q, k[src], v[src], rep.o, d_o, rep.lse, rep.delta,
                        rep.dq, rep.dk[src], rep.dv[src], rep.workspace)
    for a, b in zip(got, (rep.dq, rep.dk, rep.dv)):
        _close(a, b)
    rep.workspace.zero_()


@pytest.mark.parametrize("cp,rank,hq,hkv,d,c,batch", [(4, 0, 2, 2, 64, 128, 1), (3, 2, 4, 1, 128, 17, 2), (4, 1, 2, 2, 100, 40, 1),
                                                        (34, 5, 1, 1, 32, 9, 1)])
def test_fp32_run_equals_its_steps(cp, rank, hq, hkv, d, c, batch):
    rep, q, k, v, d_o = _replay(cp, cp, rank, hq, hkv, d, c, batch, dtype=torch.float32, code=P.FP32)
    for t in (rep.dq, rep.dk, rep.dv):
        t.fill_(9.0)
    rep.backward(q, k, v, d_o)
    got = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    for t, step in enumerate(rep.plan):
        src = step["src_rank"]
        P.attn_step_bwd(_desc(rep.shape, step, 0 if t else P.OVERWRITE_DQ), q, k[src], v[src], rep.o, d_o, rep.lse, rep.delta,
                        rep.dq, rep.dk[src], rep.dv[src])
    for a, b in zip(got, (rep.dq, rep.dk, rep.dv)):
        _close(a, b)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cp,rank,hq,hkv,c,batch", [
    (32, 0, 2, 1, 100, 1), (32, 11, 2, 1, 100, 1), (32, 31, 2, 2, 100, 2), (40, 20, 2, 1, 150, 1), (24, 3, 3, 1, 129, 1), (8, 7, 2, 1, 500, 1)])
def test_a_run_of_few_rows_shares_its_keys(cp, rank, hq, hkv, c, batch, d):
    """Row tiles whose keys, those of many chunks, several workgroups share: parts that start inside later key halves, diagonal halves, rows
    of two segments, of which one sees so little that parts of it are left without a tile, batches, two launches (40 steps)."""
    rep, q, k, v, d_o = _replay(cp, cp, rank, hq, hkv, d, c, batch)
    keys_alone = (P.StepDesc * cp)(*(_desc(rep.shape, s, P.OVERWRITE_DQ | P.BWD_ONLY_DKV) for s in rep.plan))
    assert P.workspace_bytes_steps(rep._bwd_descs) > P.workspace_bytes_steps(keys_alone)   # the partial dQ
    rep.workspace.fill_(0xA5)
    for t in (rep.dq, rep.dk, rep.dv):
        t.fill_(9.0)
    rep.backward(q, k, v, d_o)
    got = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    assert int(rep.workspace[:P.WORKSPACE_HEAD].count_nonzero()) == 0
    order = [s["src_rank"] for s in rep.plan]
    for flags in (P.OVERWRITE_DQ | P.WORKSPACE_CLEAN, P.WORKSPACE_CLEAN | P.OVERWRITE_DQ, 0):
        descs = (P.StepDesc * cp)(*(_desc(rep.shape, s, flags) for s in rep.plan))
        P.attn_steps_bwd(descs, q, [k[s] for s in order], [v[s] for s in order], None, d_o, rep.lse, rep.delta, rep.dq,
                         [rep.dk[s] for s in order], [rep.dv[s] for s in order], rep.workspace)
        assert int(rep.workspace[:P.WORKSPACE_HEAD].count_nonzero()) == 0
        if flags:
            assert all(torch.equal(a, b) for a, b in zip(got, (rep.dq, rep.dk, rep.dv)))
    _close(rep.dq, 2 * got[0])   # added to
    for t, step in enumerate(rep.plan):
        src = step["src_rank"]
        P.attn_step_bwd(_desc(rep.shape, step, P.BWD_ONLY_DQ | (0 if t else P.OVERWRITE_DQ)), q, k[src], v[src], None, d_o, rep.lse,
                        rep.delta, rep.dq, None, None)
        P.attn_step_bwd(_desc(rep.shape, step, P.BWD_ONLY_DKV), q, k[src], v[src], None, d_o, rep.lse, rep.delta, None, rep.dk[src],
                        rep.dv[src], rep.workspace)
    for a, b in zip(got, (rep.dq, rep.dk, rep.dv)):
        _close(a, b)


@pytest.mark.parametrize("cp,hq,hkv,d,c,only", [(4, 2, 2, 64, 33, 0), (8, 8, 8, 128, 640, 0), (4, 4, 1, 128, 200, P.BWD_ONLY_DQ)])
@pytest.mark.parametrize("form_delta", [True, False])
def test_a_run_that_does_not_count_leaves_its_workspace_alone(cp, hq, hkv, d, c, only, form_delta):
    rep, q, k, v, d_o = _replay(cp, cp, cp // 2, hq, hkv, d, c, 1)
    rep.backward(q, k, v, d_o)
    want = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    flags = only | P.OVERWRITE_DQ | (P.COMPUTE_DELTA if form_delta else 0)
    descs = (P.StepDesc * cp)(*(_desc(rep.shape, s, flags) for s in rep.plan))
    assert P.workspace_bytes_steps(descs) == 0
    ws = torch.full((2 * P.WORKSPACE_HEAD,), 0xA5, dtype=torch.uint8, device=DEV)
    order = [s["src_rank"] for s in rep.plan]
    P.attn_steps_bwd(descs, q, [k[s] for s in order], [v[s] for s in order], rep.o, d_o, rep.lse, rep.delta, rep.dq,
                     [rep.dk[s] for s in order], [rep.dv[s] for s in order], ws)
    assert bool((ws == 0xA5).all())
    for a, b in zip((rep.dq, rep.dk, rep.dv), want):
        _close(a, b)


@pytest.mark.parametrize("cp,rank,hq,hkv,d,c,batch", [(4, 0, 4, 4, 128, 1025, 1), (4, 0, 2, 2, 128, 1046, 2), (3, 2, 4, 2, 64, 892, 1), (40, 20, 2, 1, 64, 150, 1)])
def test_a_run_does_with_the_room_there_is(cp, rank, hq, hkv, d, c, batch):
    """Loops shared by as many workgroups as the workspace has room for, down to one and no workspace: the same sums in other orders
    (chains of some 8200 keys / 16 additions at most), counters left zero, nothing written past the room, the same bits every time."""
    rep, q, k, v, d_o = _replay(cp, cp, rank, hq, hkv, d, c, batch)
    rep.backward(q, k, v, d_o)
    want = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    full = P.workspace_bytes_steps(rep._bwd_descs)
    assert full > 0
    order = [s["src_rank"] for s in rep.plan]
    descs = (P.StepDesc * cp)(*(_desc(rep.shape, s, P.OVERWRITE_DQ | P.COMPUTE_DELTA) for s in rep.plan))
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    for room in (full - 16, full // 2 // 16 * 16, P.WORKSPACE_HEAD, 0):
        ws.fill_(0xA5)
        got = []
        for _ in range(2):
            for t in (rep.dq, rep.dk, rep.dv):
                t.fill_(9.0)
            P.attn_steps_bwd(descs, q, [k[s] for s in order], [v[s] for s in order], rep.o, d_o, rep.lse, rep.delta, rep.dq,
                             [rep.dk[s] for s in order], [rep.dv[s] for s in order], ws[:room])
            assert bool((ws[room:] == 0xA5).all())
            got.append([t.clone() for t in (rep.dq, rep.dk, rep.dv)])
        head = ws[:min(room, P.WORKSPACE_HEAD)]
        assert not bool(head.any()) or bool((head == 0xA5).all())   # (left alone where the run does not count)
        assert all(torch.equal(a, b) for a, b in zip(*got))
        for a, b in zip(got[0], want):
            _close(a, b)


def test_run_adds_to_what_is_there_and_halves_run_alone():
    rep, q, k, v, d_o = _replay(4, 2, 1, 4, 2, 64, 161, 1)
    rep.backward(q, k, v, d_o)
    want = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    order = [s["src_rank"] for s in rep.plan]
    for only in (P.BWD_ONLY_DQ, P.BWD_ONLY_DKV):
        descs = (P.StepDesc * 4)(*(_desc(rep.shape, s, only | P.binding.ACCUM_DKV) for s in rep.plan))
        ws = torch.randint(0, 255, (max(P.workspace_bytes_steps(descs), 16),), dtype=torch.uint8, device=DEV)
        P.attn_steps_bwd(descs, q, [k[s] for s in order], [v[s] for s in order], None, d_o, rep.lse, rep.delta, rep.dq,
                         [rep.dk[s] for s in order], [rep.dv[s] for s in order], ws)
    for a, b in zip((rep.dq, rep.dk, rep.dv), want):
        _close(a, 2 * b)


def test_run_without_mask():
    d, lq, lk, n = 128, 130, 333, 3
    g = torch.Generator(device=DEV).manual_seed(3)
    mk = lambda *s: (torch.randn(*s, device=DEV, generator=g) * 0.5).to(torch.float16)
    q, d_o, o, k, v = mk(1, 4, lq, d), mk(1, 4, lq, d), mk(1, 4, lq, d), mk(n, 1, 2, lk, d), mk(n, 1, 2, lk, d)
    lse, delta = torch.full((1, 4, lq), 7.0, device=DEV), torch.zeros(1, 4, lq, device=DEV)
    desc = P.make_desc(batch=1, n_q_heads=4, n_kv_heads=2, head_dim=d, q_len=lq, kv_len=lk, dtype=P.FP16, softmax_scale=d ** -0.5)
    res = []
    for run in (True, False):
        dq = torch.zeros(1, 4, lq, d, device=DEV)
        dk, dv = torch.empty(n, 1, 2, lk, d, device=DEV), torch.empty(n, 1, 2, lk, d, device=DEV)
        descs = (P.StepDesc * n)(*(desc for _ in range(n)))
        ws = torch.empty(max(P.workspace_bytes_steps(descs), P.workspace_bytes(desc), 16), dtype=torch.uint8, device=DEV)
        if run:
            P.attn_steps_bwd(descs, q, k, v, o, d_o, lse, delta, dq, dk, dv, ws)
        else:
            for t in range(n):
                P.attn_step_bwd(desc, q, k[t], v[t], o, d_o, lse, delta, dq, dk[t], dv[t], ws)
        res.append((dq, dk, dv))
    for a, b in zip(*res):
        _close(a, b)


@pytest.mark.parametrize("cp,hq,hkv,d,c", [(4, 4, 1, 128, 200), (8, 8, 8, 128, 640), (1, 2, 1, 64, 33)])
def test_a_backward_needs_nothing_of_its_workspace(cp, hq, hkv, d, c):
    """Runs with the delta (which clears the counters on the side), without it (a kernel of its own does), and the static
    scratch array, whose counters a caller cannot vouch for: all on a stream other than the workspace's, all from junk."""
    rep, q, k, v, d_o = _replay(cp, cp, cp // 2, hq, hkv, d, c, 1)
    rep.backward(q, k, v, d_o)
    want = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    order = [s["src_rank"] for s in rep.plan]
    side = torch.cuda.Stream()
    for delta in (True, False):
        for t in (rep.dq, rep.dk, rep.dv):
            t.fill_(9.0)
        rep.workspace.fill_(0xA5)
        side.wait_stream(torch.cuda.current_stream())
        if delta:
            rep.backward(q, k, v, d_o, stream=side)
        else:
            descs = (P.StepDesc * cp)(*(_desc(rep.shape, s, P.OVERWRITE_DQ) for s in rep.plan))
            P.attn_steps_bwd(descs, q, [k[s] for s in order], [v[s] for s in order], None, d_o, rep.lse, rep.delta, rep.dq,
                             [rep.dk[s] for s in order], [rep.dv[s] for s in order], rep.workspace, stream=side)
        torch.cuda.current_stream().wait_stream(side)
        assert all(torch.equal(a, b) for a, b in zip(want, (rep.dq, rep.dk, rep.dv)))
    step, src = rep.plan[0], order[0]
    res = []
    for flags in (0, P.WORKSPACE_CLEAN):
        g = [torch.empty_like(t) for t in (rep.dq, rep.dk[src], rep.dv[src])]
        P.attn_step_bwd_static(_desc(rep.shape, step, flags | P.OVERWRITE_DQ), q, k[src], v[src], None, d_o, rep.lse, rep.delta, *g)
        res.append(g)
    assert all(torch.equal(a, b) for a, b in zip(*res))


# (the last two are cut by their work: 7.2e11 operations at head_dim 64 where a launch aims at 6e11, 1.7e12 at 128 where it aims at 1.2e12)
@pytest.mark.parametrize("cp,rank,hq,hkv,d,c,batch,dtype,code", [
    (4, 2, 4, 1, 128, 200, 1, torch.bfloat16, P.BF16), (3, 0, 2, 2, 64, 33, 2, torch.float16, P.FP16), (4, 1, 2, 1, 100, 40, 1, torch.float32, P.FP32),
    (3, 1, 32, 8, 64, 2048, 1, torch.float16, P.FP16), (4, 2, 28, 4, 128, 2048, 1, torch.bfloat16, P.BF16)])
def test_strided_run_gives_the_same_bits_and_a_cut_one_the_same_sums(cp, rank, hq, hkv, d, c, batch, dtype, code):
    """Token-major q, k, v, o, d_o and dq with gaps between the rows; a run long enough for several launches against its steps."""
    rep, q, k, v, d_o = _replay(cp, cp, rank, hq, hkv, d, c, batch, dtype=dtype, code=code)
    rep.backward(q, k, v, d_o)
    want = [t.clone() for t in (rep.dq, rep.dk, rep.dv)]
    (qs, stride), (os_, _), (dos, _) = (token_major(t, 8) for t in (q, rep.o, d_o))
    ks_, vs_ = ([token_major(x, 16)[0] for x in y] for y in (k, v))
    dq, o_stride = token_major(torch.full_like(rep.dq, 5.0), 4)
    descs = (P.StepDesc * cp)(*(_desc(rep.shape, step, P.COMPUTE_DELTA | P.OVERWRITE_DQ) for step in rep.plan))
    for desc in descs:
        desc.q_stride[:], desc.kv_stride[:], desc.o_stride[:] = stride, ks_[0].stride()[:3], o_stride
    order = [s["src_rank"] for s in rep.plan]
    for t in (rep.dk, rep.dv, rep.delta):
        t.fill_(5.0)
    P.attn_steps_bwd(descs, qs, [ks_[s] for s in order], [vs_[s] for s in order], os_, dos, rep.lse, rep.delta, dq,
                     [rep.dk[s] for s in order], [rep.dv[s] for s in order], rep.workspace)
    assert all(torch.equal(a, b) for a, b in zip(want, (dq, rep.dk, rep.dv)))
    for t, step in enumerate(rep.plan):
        src = step["src_rank"]
        P.attn_step_bwd(_desc(rep.shape, step, 0 if t else P.OVERWRITE_DQ), q, k[src], v[src], None, d_o, rep.lse, rep.delta,
                        rep.dq, rep.dk[src], rep.dv[src], rep.workspace)
    longest = max(cp * 2 * c, 2 * c * hq // hkv) // 16   # additions in the longest chain: a row's keys, a key's rows
    for a, b in zip(want, (rep.dq, rep.dk, rep.dv)):
        _close(a, b, max(1e-4, 2 * longest * 2.0 ** -24))


def test_a_source_visited_twice_counts_twice():
    """The second visit writes the same dk and dv again and adds its share of dq to the first's."""
    rep, q, k, v, d_o = _replay(3, 3, 1, 4, 2, 64, 161, 1)
    plan = rep.plan
    rep.plan = [plan[1]]
    rep.backward(q, k, v, d_o)
    want = rep.dq.clone()
    rep.plan = [plan[1], plan[1]]
    rep.backward(q, k, v, d_o)
    assert torch.isfinite(rep.dk[plan[1]["src_rank"]]).all()
    _close(rep.dq, 2 * want)
