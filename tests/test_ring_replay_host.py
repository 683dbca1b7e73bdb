"""What RingReplay hands to the library, without a GPU: its buffers are on the CPU and the library's step
calls are replaced by ones that look at their arguments."""
import weakref

import pytest
import torch

import paper_2406_18485_amd as P
from paper_2406_18485_amd import binding as B
from paper_2406_18485_amd.ring import RingReplay, RingShape

CP = 4


class Recorder:
    """Stands in for the library: every step call succeeds, and `look(name, arguments)` sees it."""

    def __init__(self, look):
        self.look = look

    def __getattr__(self, name):
        def call(*args):
            self.look(name, args)
            return 0
        return call


@pytest.fixture
def replay(monkeypatch):
    """(replay, q, set of the calls made so far); `.look` may be replaced to see the arguments of a call."""
    rep = RingReplay(RingShape(cp=CP, w=2, rank=1, hq=2, hkv=1, d=64, c=8, dtype=P.BF16, scale=0.125), "cpu")
    rep.calls = []
    rep.look = lambda name, args: None

    def look(name, args):
        rep.calls.append(name)
        rep.look(name, args)
    monkeypatch.setattr(B, "lib", Recorder(look))
    return rep


def _inputs(n):
    chunks = torch.zeros(n, 1, 1, 16, 64, dtype=torch.bfloat16)
    return torch.zeros(1, 2, 16, 64, dtype=torch.bfloat16), chunks


@pytest.mark.parametrize("form", ["stacked", "list"])
@pytest.mark.parametrize("have", [1, CP - 1])
def test_too_few_chunks_are_refused_before_any_call(replay, have, form):
    q, full = _inputs(CP)
    few = full[:have] if form == "stacked" else list(full[:have])
    for k, v in ((few, full), (full, few)):
        with pytest.raises(IndexError):
            replay.forward(q, k, v)
        with pytest.raises(IndexError):
            replay.backward(q, k, v, q)
    assert not replay.calls
    replay.forward(q, full, full)
    replay.backward(q, full, full, q)
    assert replay.calls == ["loong_attn_steps_fwd", "loong_attn_steps_bwd"]


def test_chunks_made_for_the_call_live_through_it(replay):
    q, full = _inputs(CP)

    class Lazy:   # e.g. chunks kept in another form and widened when they are asked for
        def __init__(self):
            self.made = []

        def __getitem__(self, src):
            x = full[src].clone()
            self.made.append((weakref.ref(x), x.data_ptr()))
            return x

    k, v = Lazy(), Lazy()

    def look(name, args):
        for lazy, pointers in ((k, args[3]), (v, args[4])):
            assert len(lazy.made) == CP and all(ref() is not None for ref, _ in lazy.made)
            assert list(pointers) == [p for _, p in lazy.made]
    replay.look = look
    replay.forward(q, k, v)
    k.made, v.made = [], []
    replay.backward(q, k, v, q)
    assert len(replay.calls) == 2


def test_lists_may_hold_raw_pointers(replay):
    q, full = _inputs(CP)
    order = [step["src_rank"] for step in replay.plan]
    pointers = [full[src].data_ptr() for src in range(CP)]

    def look(name, args):
        assert list(args[3]) == list(args[4]) == [pointers[src] for src in order]
    replay.look = look
    replay.forward(q, pointers, pointers)
    replay.backward(q, pointers, pointers, q)
    assert len(replay.calls) == 2


def test_no_backward_vouches_for_counters_cleared_on_another_stream(replay):
    """The stream of a backward is the caller's choice, so its counters are cleared there and not at construction."""
    q, full = _inputs(CP)
    seen = []
    replay.look = lambda name, args: seen.extend(args[0][t].flags for t in range(CP))
    replay.backward(q, full, full, q)
    assert len(seen) == CP and not any(flags & P.WORKSPACE_CLEAN for flags in seen)


@pytest.mark.parametrize("fused", [True, False])
def test_changes_of_shape_and_plan_reach_the_next_call(replay, fused):
    """`shape` and `plan` are public and plain: a scale, extra flags or an order of visits set after construction count."""
    q, full = _inputs(CP)
    seen = []

    def look(name, args):
        if name == "loong_attn_step_fwd":   # one descriptor by reference, one K pointer
            seen.append((args[0]._obj.softmax_scale, args[0]._obj.flags, args[2]))
        elif name in ("loong_attn_steps_fwd", "loong_attn_steps_bwd"):
            seen.extend((args[0][t].softmax_scale, args[0][t].flags, args[3][t]) for t in range(args[1]))
    replay.look = look

    def passes():
        seen.clear()
        replay.forward(q, full, full, fuse_merge=fused)
        replay.backward(q, full, full, q)
        return list(seen)

    first = passes()
    assert len(first) == 2 * CP and {scale for scale, _, _ in first} == {0.125}
    replay.shape.scale = 0.25
    replay.shape.extra_flags = P.key_splits(2)
    assert passes() == [(0.25, flags | P.key_splits(2), k) for _, flags, k in first]
    replay.plan.reverse()
    half = replay.plan[:2]
    assert [k for _, _, k in passes()] == [k for _, _, k in first[CP - 1::-1] + first[:CP - 1:-1]]
    replay.plan = half
    assert [k for _, _, k in passes()] == [first[CP - 1][2], first[CP - 2][2]] * 2
    made = replay._fwd_descs
    passes()
    assert replay._fwd_descs is made   # nothing changed, nothing made again


def test_construction_clears_no_memory_that_calls_count_in(monkeypatch):
    """It would be cleared on the stream of the construction, at a time that calls on other streams know nothing of."""
    junk = lambda *size, **kw: torch.full(size, 0xA5 if kw["dtype"] == torch.uint8 else 7, **kw)
    monkeypatch.setattr(torch, "empty", junk)
    shape = RingShape(cp=CP, w=2, rank=1, hq=4, hkv=1, d=128, c=200, dtype=P.BF16, scale=0.125)
    rep = RingReplay(shape, "cpu")
    assert rep.workspace.numel() > B.WORKSPACE_HEAD and bool((rep.workspace == 0xA5).all())
    # a plan that asks for more: the first workspace, which another stream may be using, is kept beside the new one
    plan, rep.plan = rep.plan, rep.plan[:1]
    rep.workspace, rep._workspaces = None, []
    rep._follow()
    first, small = weakref.ref(rep.workspace), rep.workspace.numel()
    rep.plan = plan
    rep._follow()
    assert rep.workspace.numel() > small and first() is not None


def test_dq_is_zero_when_the_steps_leave_it_alone(replay):
    """Extra flags that ask for dK and dV only: dq is what no step has added to, not what the memory held."""
    q, full = _inputs(CP)
    replay.dq.fill_(7.0)
    replay.backward(q, full, full, q)
    assert bool((replay.dq == 7.0).all())    # the steps write it (here they are not the library's)
    replay.shape.extra_flags = P.BWD_ONLY_DKV
    replay.backward(q, full, full, q)
    assert bool((replay.dq == 0.0).all())


def test_a_plan_that_visits_a_source_again_runs_step_by_step(replay):
    """Two steps of a run may not share dk and dv; one after the other they may, each writing or adding in its turn."""
    q, full = _inputs(CP)
    replay.plan = [replay.plan[1], replay.plan[0], replay.plan[1]]
    seen = []

    def look(name, args):
        assert name != "loong_attn_steps_bwd"
        if name == "loong_attn_step_bwd":
            seen.append((args[0]._obj.flags & (P.COMPUTE_DELTA | P.OVERWRITE_DQ), args[2], args[9]))
    replay.look = look
    replay.backward(q, full, full, q)
    order = [step["src_rank"] for step in replay.plan]
    assert [k for _, k, _ in seen] == [full[src].data_ptr() for src in order]
    assert [dk for _, _, dk in seen] == [replay.dk[src].data_ptr() for src in order]
    assert [flags for flags, _, _ in seen] == [P.COMPUTE_DELTA | P.OVERWRITE_DQ, 0, 0]
