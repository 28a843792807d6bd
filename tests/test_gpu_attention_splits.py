"""Attention where the workgroups fill between half and all of the CUs: a request of 1024 cached keys or
more takes two key splits, a shorter one the same single split as in a small cache."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dpara_oracle as O  # noqa: E402
from paper_2609_27396_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = 2e-2  # the bf16 bar of test_gpu_parity


def _shape(nq, nkv, hd, gamma, layers=1):
    return synth.DrafterShape(n_layers=layers, hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, ffn=256,
                              vocab=1000, gamma=gamma, ar_rank=64, qk_norm=True, dtype="bf16")


# workgroups without splits: 3 x 8 KV heads x 10 query tiles = 240; 2 x 7 x 10 = 140, whose live
# workgroups do not divide by the 8 XCDs; 160 of 20 requests
@pytest.mark.parametrize("nq,nkv,hd,gamma,lens", [
    (32, 8, 64, 16, [1500, 40, 0]), (32, 8, 64, 16, [0, 1024, 1023]), (32, 8, 128, 16, [2000, 1100, 1030]),
    (28, 7, 64, 16, [10, 1600]), (8, 8, 64, 10, [0, 1200, 3, 3, 1024, 700, 1023, 2047, 0, 64] * 2)])
def test_splits_follow_each_length(nq, nkv, hd, gamma, lens):
    from paper_2609_27396_amd.harness import DeviceRound
    s = _shape(nq, nkv, hd, gamma)
    print("case splits", nq, nkv, hd, gamma, lens, file=sys.stderr, flush=True)
    wl = synth.Workload("splits", s, batch=len(lens), ctx_min=0, ctx_max=0, p_reject=0.3, seed_in=7)
    w = synth.make_weights(s, seed=3, gain_jitter=0.1)
    ri = synth.make_round(wl, ctx_lens=lens)
    dr = DeviceRound(s, w, ri, ctx_cap=2176)
    dr.backbone()
    assert dr.status() == 0
    for b in range(min(len(lens), 10)):
        ref = O.backbone_all_boundaries(s, w, ri.ctx_feats[b], ri.spine[b], "bf16")["reps"]
        assert np.abs(dr.reps[b].cpu().numpy() - ref).max() <= TOL, b
    # the same keys in a cache of fewer than 1024: one split for all
    cap = 960
    small = [min(n, cap - gamma - 1) for n in lens]
    ds = DeviceRound(s, w, synth.make_round(wl, ctx_lens=small), ctx_cap=cap, drafter=dr.d)
    ds.ctx.k.copy_(dr.ctx.k[:, :, :, :cap])
    ds.ctx.v.copy_(dr.ctx.v[..., :cap])
    ds.spine.copy_(dr.spine)
    ds.backbone()
    assert ds.status() == 0
    for b, (n, m) in enumerate(zip(lens, small)):
        if n == m:
            assert torch.equal(dr.reps[b], ds.reps[b]), b
