"""Workgroups of the multi-trial kernel take their items as they need them (beyond two items each, of operand faults
beyond four; from 64 on also other XCDs'): every item is computed once, whichever workgroup takes it.  Against the
one-trial kernel, byte for byte.  Each test works out from the sizes that its launches do take them so."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu

SHAPE = {0: (1, 256, 256, 1), 1: (1, 128, 128, 2), 3: (4, 128, 128, 1), 4: (2, 128, 128, 1), 5: (8, 128, 64, 1), 6: (8, 64, 64, 2)}


def _rounds(cfg, M, N, part, n):
    """Items per workgroup of a launch over `part` of n trials: trials per item, tile, workgroups per CU by configuration."""
    import torch
    R, bm, bn, wgs = SHAPE[cfg]
    tiles = -(-M // bm) * -(-N // bn)
    places = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8 * wgs
    return tiles * -(-part // R) / min(places, tiles * -(-n // R))


def _faults(plan, n):
    f = fi.fi_sample_faults(3, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    f[2::5] = fi.fi_sample_faults(4, 0, n, plan.desc, fi.KIND_ALL_B, 2)[2::5]
    f[3::5] = fi.fi_sample_faults(5, 0, n, plan.desc, fi.KIND_ALL_PRODUCT, 4)[3::5]
    f[7]["kind"] = 0
    return f


# K = 128 is the shortest item that takes its successor so, K = 192 has an odd number of k-tiles
@pytest.mark.parametrize("M,N,K,n,cfg", [(70, 60, 128, 17000, 6), (70, 60, 192, 17000, 6), (64, 130, 128, 16384, 6),
                                         (600, 300, 128, 6000, 6), (130, 70, 320, 4400, 5), (257, 300, 128, 520, 4),
                                         (300, 500, 128, 800, 3), (300, 500, 192, 800, 3)])
def test_campaign_items_are_taken_once(M, N, K, n, cfg):
    Aw, Bw = wl.gaussian(M, N, K, orc.FP16, seed=M + K)
    one, plan = gu.make_plan(Aw, Bw, 32, orc.FP16, cfg=2), gu.make_plan(Aw, Bw, 32, orc.FP16, cfg=cfg)
    faults = _faults(plan, n)
    operand = int(np.isin(faults["kind"], (fi.SITE_A, fi.SITE_B)).sum())
    assert _rounds(cfg, M, N, n - operand, n) > 2 and _rounds(cfg, M, N, operand, n) > 4
    want = gu.gpu_campaign(one, faults, wl.CORRECT_RECOMPUTE)
    for _ in range(2):
        got = gu.gpu_campaign(plan, faults, wl.CORRECT_RECOMPUTE)
        assert got.tobytes() == want.tobytes(), [t for t in range(n) if got[t] != want[t]][:5]
    one.destroy()
    plan.destroy()


# one launch has all the work: workgroups look for items in the other XCDs' slices when theirs is used up
@pytest.mark.parametrize("kind", [fi.KIND_ALL_ACC, fi.KIND_ALL_A, fi.KIND_ALL_B])
@pytest.mark.parametrize("M,N,K,n,cfg", [(600, 300, 128, 6000, 6), (600, 290, 192, 4400, 3)])
def test_items_of_other_slices_are_taken_once(M, N, K, n, cfg, kind):
    Aw, Bw = wl.gaussian(M, N, K, orc.BF16, seed=N)
    one, plan = gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=2), gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=cfg)
    faults = fi.fi_sample_faults(11, 0, n, plan.desc, kind, 1)
    assert _rounds(cfg, M, N, n, n) > 64
    want = gu.gpu_campaign(one, faults, wl.CORRECT_ZERO)
    got = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    assert got.tobytes() == want.tobytes(), [t for t in range(n) if got[t] != want[t]][:5]
    one.destroy()
    plan.destroy()


# 128 x 128 tiles (cfg 1, 512 workgroups) and 256 x 256 (cfg 0, 256): a few items each, many, and so few trials that
# the counters have no room; the site words, which hold the counters meanwhile, are 0 afterwards
@pytest.mark.parametrize("M,N,K,n,cfg,rounds", [(100, 128, 128, 1100, 1, 2), (40, 30, 192, 33000, 1, 64), (300, 200, 128, 700, 1, 8),
                                                (260, 200, 128, 300, 0, 2), (1500, 1500, 128, 7, 1, 0), (1500, 1500, 128, 8, 1, 2)])
def test_next_layer_items_are_taken_once(M, N, K, n, cfg, rounds):
    import torch
    assert _rounds(cfg, M, N, n, n) > rounds
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
