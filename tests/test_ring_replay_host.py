"""What RingReplay hands to the library, without a GPU: its buffers are on the CPU and the library's step
calls are replaced by ones that look at their arguments."""
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
