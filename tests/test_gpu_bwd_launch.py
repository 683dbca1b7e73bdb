"""The backward step as one launch: what it clears, writes and leaves behind besides the gradients that
the parity tests compare (dq written instead of added to, keys nobody sees, the workspace's counters)."""
import math

import pytest
import torch

import paper_2406_18485_amd as P
from gpu_harness import DEV, workspace_for

pytestmark = pytest.mark.gpu

TORCH = {P.BF16: torch.bfloat16, P.FP16: torch.float16, P.FP32: torch.float32}


def _step(dtype, hq, hkv, d, c, q_chunk, kv_chunk, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    mk = lambda h: (torch.randn(1, h, 2 * c, d, generator=g) * 0.5).to(TORCH[dtype]).to(DEV)
    t = dict(q=mk(hq), k=mk(hkv), v=mk(hkv), d_o=mk(hq))
    t["lse"] = (torch.rand(1, hq, 2 * c, generator=g) + math.log(2 * c)).to(DEV)
    t["lse"][0, 0, 0] = -math.inf   # a row that takes no part
    t["delta"] = torch.randn(1, hq, 2 * c, generator=g).to(DEV) * 0.1
    desc = lambda flags: P.make_desc(batch=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, q_len=2 * c, kv_len=2 * c, dtype=dtype,
                                     softmax_scale=1 / math.sqrt(d), causal=True, chunk_len=c, q_chunk=q_chunk,
                                     kv_chunk=kv_chunk, flags=flags)
    return t, desc


def _run(t, desc, dq, workspace):
    dk, dv = torch.full(t["k"].shape, 7.0, device=DEV), torch.full(t["k"].shape, 7.0, device=DEV)
    P.attn_step_bwd(desc, t["q"], t["k"], t["v"], None, t["d_o"], t["lse"], t["delta"], dq, dk, dv, workspace)
    torch.cuda.synchronize()
    return dq, dk, dv


STEPS = [((1, 6), (1, 6)), ((1, 6), (0, 7)), ((1, 6), (3, 4))]   # diagonal; late keys unseen; early rows blind


@pytest.mark.parametrize("chunks", STEPS)
@pytest.mark.parametrize("dtype,hq,hkv,d,c", [
    (P.BF16, 4, 1, 128, 200), (P.BF16, 2, 2, 64, 33), (P.FP16, 3, 1, 128, 129), (P.BF16, 8, 8, 128, 1024), (P.FP32, 2, 1, 64, 65)])
def test_overwritten_dq_and_cleared_gradients(dtype, hq, hkv, d, c, chunks):
    t, desc = _step(dtype, hq, hkv, d, c, *chunks, seed=c)
    ws = workspace_for(desc(0))
    ws.fill_(0xA5)   # anything may be in it
    want = _run(t, desc(0), torch.zeros(t["q"].shape, device=DEV), ws)
    got = _run(t, desc(P.OVERWRITE_DQ), torch.full(t["q"].shape, 3.0, device=DEV), ws)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert float(got[0][0, 0, 0].abs().max()) == 0.0
    if chunks[1] == (0, 7):
        assert float(got[1][:, :, c:].abs().max()) == 0.0 and float(got[2][:, :, c:].abs().max()) == 0.0
    if chunks[1] == (3, 4):
        assert float(got[0][:, :, :c].abs().max()) == 0.0


@pytest.mark.parametrize("hq,hkv,d,c,chunks,shared", [
    (4, 1, 128, 200, STEPS[1], True), (4, 1, 64, 777, STEPS[0], True), (8, 8, 128, 1024, STEPS[1], True), (8, 8, 128, 2048, STEPS[2], False)])
def test_counters_stay_zero_between_calls(hq, hkv, d, c, chunks, shared):
    t, desc = _step(P.BF16, hq, hkv, d, c, *chunks, seed=d + c)
    need = P.workspace_bytes(desc(0))
    assert (need > 0) == shared
    head = P.WORKSPACE_HEAD
    ws = torch.zeros(max(need, 16), dtype=torch.uint8, device=DEV)
    junk = torch.full_like(ws, 0xFF)
    want = _run(t, desc(0), torch.zeros(t["q"].shape, device=DEV), junk)
    for _ in range(3):
        got = _run(t, desc(P.WORKSPACE_CLEAN), torch.zeros(t["q"].shape, device=DEV), ws)
        assert int(ws[:head].count_nonzero()) == 0
        for a, b in zip(got, want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("word", [0x70000000, 0xA5A5A5A5 - (1 << 32), -1 - 100])
def test_counters_past_the_last_arrival_give_nan(word):
    """Counters that a caller vouched for and did not clear: no workgroup waits for another, the tiles say that something is
    wrong, and the next call, which clears its counters, is right again."""
    t, desc = _step(P.BF16, 4, 1, 128, 200, *STEPS[0], seed=3)
    ws = workspace_for(desc(0))
    want = _run(t, desc(0), torch.zeros(t["q"].shape, device=DEV), ws)
    ws[:P.WORKSPACE_HEAD].view(torch.int32).fill_(word)
    got = _run(t, desc(P.WORKSPACE_CLEAN), torch.zeros(t["q"].shape, device=DEV), ws)
    assert torch.equal(got[0], want[0]) and torch.isnan(got[1]).all() and torch.isnan(got[2]).all()
    again = _run(t, desc(0), torch.zeros(t["q"].shape, device=DEV), ws)
    assert all(torch.equal(a, b) for a, b in zip(again, want))


def _many(n, batch, d=64):
    """One query and one key per batch element, n steps that share them: a workgroup each in either half."""
    g = torch.Generator(device=DEV).manual_seed(n)
    mk = lambda: torch.randn(batch, 1, 1, d, device=DEV, generator=g, dtype=torch.bfloat16) * 0.5
    q, k, v, d_o = mk(), mk(), mk(), mk()
    lse, delta = torch.zeros(batch, 1, 1, device=DEV), torch.zeros(batch, 1, 1, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    dq, dk, dv = torch.full((batch, 1, 1, d), 5.0, **f32), torch.empty(n, batch, 1, 1, d, **f32), torch.empty(n, batch, 1, 1, d, **f32)
    descs = (P.StepDesc * n)(*(P.make_desc(batch=batch, n_q_heads=1, n_kv_heads=1, head_dim=d, q_len=1, kv_len=1, dtype=P.BF16,
                                           softmax_scale=0.125, flags=P.OVERWRITE_DQ) for _ in range(n)))
    return descs, q, k, v, d_o, lse, delta, dq, dk, dv


@pytest.mark.parametrize("n,batch", [(1, 1 << 22), (32, 1 << 18)])
def test_more_workgroups_than_one_launch_takes(n, batch):
    """A launch takes fewer than 2^32 threads, 2^23 workgroups of 512: the two halves of the first case have that many together,
    the key tiles of the second's 32 steps alone.  With one key P = exp(scale q.k - lse), dS = P (dO.v - delta)."""
    descs, q, k, v, d_o, lse, delta, dq, dk, dv = _many(n, batch)
    ws = torch.empty(max(P.workspace_bytes_steps(descs), 16), dtype=torch.uint8, device=DEV)
    P.attn_steps_bwd(descs, q, [k] * n, [v] * n, None, d_o, lse, delta, dq, dk, dv, ws)
    torch.cuda.synchronize()
    for part in (slice(0, 1 << 16), slice(batch // 2, batch // 2 + (1 << 16)), slice(batch - (1 << 16), batch)):
        qf, kf, vf, of = (t[part].float() for t in (q, k, v, d_o))
        p = torch.exp((qf * kf).sum(-1, keepdim=True) * 0.125)
        ds = p * (of * vf).sum(-1, keepdim=True) * 0.125
        for t in {0, n - 1}:
            # P, dS and the scaled operand of the exponent are rounded to 8 bits: 2^-9 each, products of size one
            assert float((dv[t, part] - p * of).abs().max()) < 2e-2 and float((dk[t, part] - ds * qf).abs().max()) < 2e-2
        assert float((dq[part] - n * ds * kf).abs().max()) < n * 2e-2


def test_a_step_too_large_for_a_launch_is_refused_before_anything_runs():
    (desc,), q, k, v, d_o, lse, delta, dq, dk, dv = _many(1, 1 << 23)
    desc.flags |= P.COMPUTE_DELTA
    delta.fill_(3.0)
    with pytest.raises(P.LoongError) as e:
        P.attn_step_bwd(desc, q, k, v, q, d_o, lse, delta, dq, dk[0], dv[0])
    torch.cuda.synchronize()
    assert e.value.code == P.E_UNSUPPORTED and bool((delta == 3.0).all()) and bool((dq == 5.0).all())
    with pytest.raises(P.LoongError) as e:
        P.attn_step_fwd(desc, q, k, v, dq, lse)
    torch.cuda.synchronize()
    assert e.value.code == P.E_UNSUPPORTED and bool((dq == 5.0).all())


@pytest.mark.parametrize("dtype", [P.BF16, P.FP16])
@pytest.mark.parametrize("lq,lk,hq,hkv", [(1, 1, 1, 1), (31, 129, 2, 1), (64, 64, 1, 1), (65, 127, 4, 2), (200, 700, 3, 1), (513, 257, 8, 8)])
@pytest.mark.parametrize("ks", [1, 2, 4])
@pytest.mark.parametrize("per_unit", [1, 2])
def test_head_dim_64_gradients_at_the_edges_of_tiles(lq, lk, hq, hkv, ks, dtype, per_unit):
    """One workgroup per unit, and (as many copies of the problem as fill the chip) two: offsets formed once per query row (rows past the end and rows with LSE = -inf give nothing),
    starting values spread by the matrix cores (a row with an LSE and a delta beyond the half's range among them), tiles two and
    four deep.  Against fp64 from the same LSE and delta; the bound is what rounding P, dS, K and Q to 16 bits leaves: about 2^-9
    (2^-12) of the terms' root sum of squares, eight times that for the largest of some 1e5 values."""
    g = torch.Generator(device="cpu").manual_seed(lq * 7 + lk)
    mk = lambda h, n: (torch.randn(1, h, n, 64, generator=g) * 0.5).to(TORCH[dtype])
    q, k, v, d_o = mk(hq, lq), mk(hkv, lk), mk(hkv, lk), mk(hq, lq)
    x = lambda t: t.double().repeat_interleave(hq // t.shape[1], 1)
    s = (x(q) @ x(k).transpose(-1, -2)) * 0.125
    lse = torch.logsumexp(s, -1).float()
    p = torch.exp(s - lse.double()[..., None])
    delta = (x(d_o) * (p @ x(v))).sum(-1).float()
    if lq > 1:
        lse[0, 0, 0], lse[0, -1, -1], delta[0, -1, -1] = -math.inf, 1e6, -1e6   # no key at all; probabilities of zero
        p[0, 0, 0], p[0, -1, -1] = 0.0, 0.0
    ds = p * (x(d_o) @ x(v).transpose(-1, -2) - delta.double()[..., None]) * 0.125
    group = lambda t: t.reshape(1, hkv, hq // hkv, lk, 64).sum(2)
    want = ds @ x(k), group(ds.transpose(-1, -2) @ x(q)), group(p.transpose(-1, -2) @ x(d_o))
    terms = (ds.abs().square() @ x(k).square()).sqrt(), group(ds.square().transpose(-1, -2) @ x(q).square()).sqrt(), group(
        p.square().transpose(-1, -2) @ x(d_o).square()).sqrt()
    batch = 1 if per_unit == 1 else -(-300 // (hkv * -(-lk // 128)))   # (more than 288 workgroups over keys alone)
    desc = P.make_desc(batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=64, q_len=lq, kv_len=lk, dtype=dtype, softmax_scale=0.125,
                       flags=P.key_splits(ks))
    t = dict(q=q, k=k, v=v, d_o=d_o, lse=lse, delta=delta)
    t = {n: x.expand(batch, *x.shape[1:]).contiguous().to(DEV) for n, x in t.items()}
    got = _run(t, desc, torch.zeros(t["q"].shape, device=DEV), workspace_for(desc))
    for a in got:   # the copies are one result
        assert torch.equal(a, a[:1].expand_as(a))
    got = [a[:1] for a in got]
    eps = 2.0 ** (-9 if dtype == P.BF16 else -12)
    for a, b, scale in zip(got, want, terms):
        err = (a.cpu().double() - b).abs()
        assert bool((err <= 8 * eps * (scale + scale.max() / 8) + 1e-6).all()), float((err / (scale + scale.max() / 8) / eps).max())


@pytest.mark.parametrize("batch", [1, 300])   # one and two workgroups per unit
@pytest.mark.parametrize("ks", [1, 4])
@pytest.mark.parametrize("most", [3.4e38, 3.4028234663852886e38])
def test_the_largest_floats_are_no_infinities(batch, ks, most):
    """head_dim 64: a row whose probabilities are zero (an LSE of 1e6) and whose delta is the largest float takes no part, and an LSE of the
    lowest float, on the diagonal, means what -inf means."""
    g = torch.Generator(device=DEV).manual_seed(ks)
    mk = lambda: (torch.randn(1, 1, 64, 64, generator=g, device=DEV) * 0.5).to(torch.bfloat16).expand(batch, -1, -1, -1).contiguous()
    t = dict(q=mk(), k=mk(), v=mk(), d_o=mk(), lse=torch.full((batch, 1, 64), 4.0, device=DEV), delta=torch.zeros(batch, 1, 64, device=DEV))
    t["lse"][:, 0, 5:7] = 1e6
    t["lse"][:, 0, 40] = -math.inf
    desc = P.make_desc(batch=batch, n_q_heads=1, n_kv_heads=1, head_dim=64, q_len=64, kv_len=64, dtype=P.BF16, softmax_scale=0.125,
                       causal=True, chunk_len=32, q_chunk=(0, 1), kv_chunk=(0, 1), flags=P.key_splits(ks))
    zeros = lambda: torch.zeros(t["q"].shape, device=DEV)
    want = _run(t, desc, zeros(), workspace_for(desc))
    t["delta"][:, 0, 5], t["delta"][:, 0, 6] = most, -most
    got = _run(t, desc, zeros(), workspace_for(desc))
    assert all(torch.equal(a, b) for a, b in zip(got, want)) and float(got[0][:, 0, 5:7].abs().max()) == 0.0
    t["lse"][:, 0, 40] = -3.4028234663852886e38
    got = _run(t, desc, zeros(), workspace_for(desc))
    assert all(torch.equal(a, b) for a, b in zip(got[1:], want[1:]))


@pytest.mark.parametrize("dtype", [P.BF16, P.FP16])
@pytest.mark.parametrize("lq,lk", [(1, 1), (33, 129), (64, 700), (63, 128)])
@pytest.mark.parametrize("ks", [1, 2, 4])
def test_either_form_at_head_dim_64_gives_the_same_bits(lq, lk, ks, dtype):
    """One problem of few workgroups and 300 copies of it, which fill the chip twice: dQ alone, dK/dV alone and both.  (One query tile,
    so that no loop is shared in either.)"""
    g = torch.Generator(device=DEV).manual_seed(lq + lk)
    mk = lambda n: (torch.randn(1, 1, n, 64, generator=g, device=DEV) * 0.5).to(TORCH[dtype])
    one = dict(q=mk(lq), k=mk(lk), v=mk(lk), d_o=mk(lq), lse=torch.full((1, 1, lq), math.log(lk) + 0.1, device=DEV),
               delta=torch.randn(1, 1, lq, generator=g, device=DEV) * 0.1)
    for flags in (0, P.BWD_ONLY_DQ, P.BWD_ONLY_DKV):
        res = []
        for batch in (1, 300):
            desc = P.make_desc(batch=batch, n_q_heads=1, n_kv_heads=1, head_dim=64, q_len=lq, kv_len=lk, dtype=dtype, softmax_scale=0.125,
                               flags=flags | P.key_splits(ks))
            assert P.workspace_bytes(desc) == 0
            t = {n: x.expand(batch, *x.shape[1:]).contiguous() for n, x in one.items()}
            res.append(_run(t, desc, torch.zeros(t["q"].shape, device=DEV), None))
        for a, b in zip(*res):
            assert torch.equal(a.expand_as(b), b)


@pytest.mark.parametrize("lq,lk,hq,hkv,parts", [(4096, 4096, 8, 8, 1), (3072, 8192, 8, 4, 1), (8192, 2048, 8, 8, 2)])
def test_a_step_that_could_fill_the_chip_does_without_the_room_for_it(lq, lk, hq, hkv, parts):
    """head_dim 64: with a workspace of the reported size the query loops are split until the chip is full, with a smaller one only until
    every unit has a workgroup (`parts` per key tile), which takes less or none.  The same sums in another order: dk and dv are chains of
    lq hq / hkv / 16 <= 512 additions, so two orders differ by at most 2 * 512 * 2^-24 = 6.1e-5 of the largest running sum."""
    g = torch.Generator(device=DEV).manual_seed(lq + lk)
    mk = lambda h, n: (torch.randn(1, h, n, 64, generator=g, device=DEV) * 0.5).to(torch.bfloat16)
    t = dict(q=mk(hq, lq), k=mk(hkv, lk), v=mk(hkv, lk), d_o=mk(hq, lq))
    t["lse"], t["delta"] = torch.full((1, hq, lq), math.log(lk) + 0.1, device=DEV), torch.zeros(1, hq, lq, device=DEV)
    desc = P.make_desc(batch=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=64, q_len=lq, kv_len=lk, dtype=P.BF16, softmax_scale=0.125,
                       flags=P.OVERWRITE_DQ)
    dq = lambda: torch.full(t["q"].shape, 3.0, device=DEV)
    least = 0 if parts == 1 else P.WORKSPACE_HEAD + -(-lk // 128) * hkv * parts * 65536
    full = P.workspace_bytes(desc)
    assert full > least
    want = _run(t, desc, dq(), torch.full((full,), 0xA5, dtype=torch.uint8, device=DEV))
    small = torch.full((full - 16,), 0xA5, dtype=torch.uint8, device=DEV)
    for ws in [small, small[:least]] + ([None] if least == 0 else []):
        got = _run(t, desc, dq(), ws)
        for a, b in zip(got, want):
            assert float((a - b).abs().max()) <= 1e-4 * float(b.abs().max())
    if least == 0:
        assert bool((small == 0xA5).all())
    else:
        for ws, code in ((small[:least - 16], P.E_SHAPE), (None, P.E_NULL)):
            with pytest.raises(P.LoongError) as e:
                _run(t, desc, dq(), ws)
            assert e.value.code == code


@pytest.mark.parametrize("dtype", [P.BF16, P.FP16])
@pytest.mark.parametrize("d,lq,lk,hq,hkv,ks", [(64, 33, 3500, 2, 1, 0), (128, 121, 6001, 4, 2, 0), (128, 1, 2000, 1, 1, 1), (64, 300, 1700, 3, 3, 2), (128, 64, 3073, 2, 2, 4)])
def test_keys_of_a_row_tile_shared_by_several_workgroups(d, lq, lk, hq, hkv, ks, dtype):
    """Few rows, many keys: partial dQ through the workspace, added up in order.  Against the dQ half alone (which shares nothing)
    within fp32 sums in another order (some 400 additions, each off by at most 2^-24 of the running sum to either side: 20 of them add up, 2.5
times that for the largest of 1e5 values); counters left zero; dq written and added to; the same bits every time."""
    g = torch.Generator(device="cpu").manual_seed(lq + lk)
    mk = lambda h, n: (torch.randn(1, h, n, d, generator=g) * 0.5).to(TORCH[dtype]).to(DEV)
    t = dict(q=mk(hq, lq), k=mk(hkv, lk), v=mk(hkv, lk), d_o=mk(hq, lq))
    t["lse"] = torch.full((1, hq, lq), math.log(lk) + 0.1, device=DEV)
    t["delta"] = torch.randn(1, hq, lq, generator=g).to(DEV) * 0.01
    desc = lambda flags: P.make_desc(batch=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, q_len=lq, kv_len=lk, dtype=dtype,
                                     softmax_scale=d ** -0.5, flags=flags | P.key_splits(ks))
    need = P.workspace_bytes(desc(0))
    assert need > P.workspace_bytes(desc(P.BWD_ONLY_DKV))   # the partial dQ
    alone = _run(t, desc(P.BWD_ONLY_DQ | P.OVERWRITE_DQ), torch.full(t["q"].shape, 3.0, device=DEV), None)[0]
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device=DEV)
    first = _run(t, desc(P.OVERWRITE_DQ), torch.full(t["q"].shape, 3.0, device=DEV), ws)
    assert int(ws[:P.WORKSPACE_HEAD].count_nonzero()) == 0
    scale = float(alone.abs().max())
    assert float((first[0] - alone).abs().max()) <= 3e-6 * scale
    again = _run(t, desc(0), first[0].clone(), ws)
    assert float((again[0] - 2 * alone).abs().max()) <= 6e-6 * scale and torch.equal(again[1], first[1]) and torch.equal(again[2], first[2])
    for _ in range(3):
        more = _run(t, desc(P.OVERWRITE_DQ), torch.full(t["q"].shape, 3.0, device=DEV), ws)
        assert all(torch.equal(a, b) for a, b in zip(more, first))
