"""The fp32-storage kernels at the edges of their tiles: 16-row and 16-key tiles, 32-row workgroups, head
dimensions the matrix instruction's blocks do not divide, loops shorter than the waves that share them."""
import math

import numpy as np
import pytest
import torch

import paper_2406_18485_amd as P
from gpu_harness import DEV, Replayed, check_full, oracle_full
from workloads import RingConfig, make_inputs

pytestmark = pytest.mark.gpu


# (the last two have 32-row workgroups: at least two for every one of 256 units)
@pytest.mark.parametrize("hq,hkv,d,c", [(1, 1, 4, 1), (2, 1, 20, 7), (3, 3, 32, 16), (2, 2, 60, 17), (4, 1, 64, 33), (6, 2, 68, 15),
                                        (1, 1, 100, 129), (2, 1, 124, 48), (8, 2, 128, 31), (32, 8, 32, 257), (16, 4, 100, 528)])
def test_every_tile_edge_against_the_oracle(hq, hkv, d, c):
    """fp32 sums of at most 4 c + d terms of size one: 1e-5 of the largest value, far inside 2e-4."""
    cfg = RingConfig("fp32_edges", cp=2, w=2, rank=1, hq=hq, hkv=hkv, d=d, c=c, dtype="fp32", sigma=1.0, seed=d + c)
    inp = make_inputs(cfg)
    check_full(Replayed(cfg, inp).run(), oracle_full(cfg, inp), tol_o=2e-4, tol_lse=1e-4)


@pytest.mark.parametrize("d,c,at", [(32, 40, 17), (64, 23, 20), (100, 16, 9), (128, 33, 30)])
@pytest.mark.parametrize("bad", [math.inf, math.nan])
def test_values_behind_the_mask_stay_out(d, c, at, bad):
    """Rows before token `at` of the diagonal blocks do not see it and keys after it are not seen by it: an infinity
    there leaves their results what they are without it.  (Tiles that hold one add their products in another order: sums of
    n <= 80 terms w x with sum |w x| < 20 move by less than n 2^-24 20 = 1e-4.)"""
    same = lambda a, b: float((a - b).abs().max()) < 1e-4   # false for infinities and NaN
    rng = np.random.default_rng(c)
    mk = lambda: torch.from_numpy(rng.standard_normal((1, 1, 2 * c, d)).astype(np.float32)).to(DEV)
    q, k, v, d_o = mk(), mk(), mk(), mk()
    desc = P.make_desc(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d, q_len=2 * c, kv_len=2 * c, dtype=P.FP32, softmax_scale=d ** -0.5,
                       causal=True, chunk_len=c, q_chunk=(0, 3), kv_chunk=(0, 3), flags=P.COMPUTE_DELTA)

    def run(k, v, d_o, forward=None):
        out, lse = torch.empty(1, 1, 2 * c, d, device=DEV), torch.empty(1, 1, 2 * c, device=DEV)
        P.attn_step_fwd(desc, q, k, v, out, lse)
        o, l = forward or (out, lse)
        g = [torch.zeros(1, 1, 2 * c, d, device=DEV) for _ in range(3)]
        P.attn_step_bwd(desc, q, k, v, o, d_o, l, torch.empty_like(lse), *g)
        torch.cuda.synchronize()
        return out, lse, *g

    good = run(k, v, d_o)
    k2, v2, d_o2 = k.clone(), v.clone(), d_o.clone()
    k2[..., at, 1] = bad
    v2[..., at, 2] = bad
    got = run(k2, v2, d_o, forward=good[:2])
    for a, b in zip(got[:3], good[:3]):   # out, lse, dq of the rows that do not see the key
        assert same(a[:, :, :at], b[:, :, :at])
    assert not torch.isfinite(got[0][:, :, at]).all()
    d_o2[..., c + at, 3] = bad            # a row of the second half: keys of that half after it are not seen by it
    got = run(k, v, d_o2, forward=good[:2])
    for a, b in zip(got[3:], good[3:]):
        assert same(a[:, :, c + at + 1:], b[:, :, c + at + 1:])
        assert not torch.isfinite(a[:, :, :at]).all()
