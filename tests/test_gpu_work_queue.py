"""Workgroups of the multi-trial kernel take their items as they need them (more than two items each; from 64
on also other XCDs'): every item is computed once, whichever workgroup takes it.  Against the one-trial kernel,
byte for byte."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def _faults(plan, n):
    f = fi.fi_sample_faults(3, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    f[2::5] = fi.fi_sample_faults(4, 0, n, plan.desc, fi.KIND_ALL_B, 2)[2::5]
    f[3::5] = fi.fi_sample_faults(5, 0, n, plan.desc, fi.KIND_ALL_PRODUCT, 4)[3::5]
    f[7]["kind"] = 0
    return f


# items per workgroup: the 64 x 64 shape (cfg 6) has 512 workgroups, eight trials an item; K = 128 is the shortest
# item that takes its successor so, K = 192 has an odd number of k-tiles
@pytest.mark.parametrize("M,N,K,n,cfg", [(70, 60, 128, 4200, 6), (70, 60, 192, 4080, 6), (64, 130, 128, 16384, 6),
                                         (600, 300, 128, 6000, 6), (130, 70, 320, 3000, 5), (257, 300, 128, 520, 4),
                                         (300, 500, 128, 270, 3)])
def test_campaign_items_are_taken_once(M, N, K, n, cfg):
    Aw, Bw = wl.gaussian(M, N, K, orc.FP16, seed=M + K)
    one, plan = gu.make_plan(Aw, Bw, 32, orc.FP16, cfg=2), gu.make_plan(Aw, Bw, 32, orc.FP16, cfg=cfg)
    faults = _faults(plan, n)
    want = gu.gpu_campaign(one, faults, wl.CORRECT_RECOMPUTE)
    for _ in range(2):
        got = gu.gpu_campaign(plan, faults, wl.CORRECT_RECOMPUTE)
        assert got.tobytes() == want.tobytes(), [t for t in range(n) if got[t] != want[t]][:5]
    one.destroy()
    plan.destroy()


# 128 x 128 tiles (cfg 1, 512 workgroups) and 256 x 256 (cfg 0, 256): a few items each, many, and so few trials that
# the counters have no room; the site words, which hold the counters meanwhile, are 0 afterwards
@pytest.mark.parametrize("M,N,K,n,cfg", [(100, 128, 128, 1100, 1), (40, 30, 192, 33000, 1), (300, 200, 128, 700, 1),
                                         (260, 200, 128, 300, 0), (1500, 1500, 128, 7, 1), (1500, 1500, 128, 8, 1)])
def test_next_layer_items_are_taken_once(M, N, K, n, cfg):
    import torch
    Aw, Bw = wl.gaussian(M, N, K, orc.BF16, seed=M + K)
    one, plan = gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=2), gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=cfg)
    rng = np.random.default_rng(n)
    a = torch.from_numpy(Aw.view(np.int16).copy()).cuda()
    stack = a.expand(n, M, K).clone()
    for t in rng.choice(n, size=min(n, 300), replace=False):
        stack[int(t), int(rng.integers(M)), int(rng.integers(K))] ^= int(1 << rng.integers(15))
    stack[n // 2, M - 1, K - 1] = 0x7F80                 # an Inf
    want, got = fi.empty_results(n), fi.empty_results(n)
    one.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_ZERO, want)
    for _ in range(2):
        got.fill_(0xAB)
        plan.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_ZERO, got)
        g, w = fi.results_to_host(got)[:n], fi.results_to_host(want)[:n]
        assert g.tobytes() == w.tobytes(), [t for t in range(n) if g[t] != w[t]][:5]
    assert not g["site_word_before"].any() and not g["site_word_after"].any() and g["n_flagged"].any()
    one.destroy()
    plan.destroy()
