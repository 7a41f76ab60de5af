"""Batches that run one wave per (trial, 32 x 32 tile) - on the smallest problems one workgroup per
trial - against the multi-trial kernel on the same faults: records and outputs have to be the same bytes (the same sequence of matrix steps)."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu
from test_gpu_affected import _faults

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 1, 16, 16),          # one step, one element
    (33, 31, 48, 16),        # a ragged k-tile alone, tiles ragged both ways
    (64, 96, 64, 32),        # whole tiles, one k-tile
    (65, 129, 208, 16),      # strips of 4, 2 and 1 tiles all ragged; more k-tiles than buffers
    (32, 40, 1008, 16),      # many k-tiles, the last ragged
    (100, 128, 128, 32),     # one workgroup per trial unless outputs are stored: all 16 waves, 2 k-tiles
    (512, 20, 80, 16),       # the same, one column of 16 tiles, ragged k-tile
])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 40])        # 1, 2 and 4 trials per workgroup, padded groups
@pytest.mark.parametrize("fmt", [orc.FP16, orc.BF16])
def test_small_batches_equal_the_multi_trial_kernel(shape, n, fmt):
    import torch
    M, N, K, kb = shape
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=M + N + K)
    wide = np.full((N, K + 8), 0x7FFF, np.uint16)       # rows of B longer than K, the gap full of NaN
    wide[:, :K] = Bw
    d_A, d_B = fi.words_to_device(Aw), fi.words_to_device(wide)
    for policy, check in ((wl.CORRECT_ZERO, fi.PCHECK_RANGE_MAX), (wl.CORRECT_RECOMPUTE, fi.PCHECK_NONE),
                          (wl.CORRECT_NONE, fi.PCHECK_BOUND)):
        bound = (fi.BOUND_EXPONENT, fi.BOUND_ROWCOL, fi.BOUND_GLOBAL)[policy]
        got = []
        for cfg in (-1, 6):                             # the library's choice; eight trials on 64 x 64 tiles
            plan = fi.Plan(fi.plan_desc(M, N, K, kb, fmt, bound_mode=bound, ldb=K + 8), d_A, d_B)
            plan.tune(cfg)
            plan.set_product_check(check)
            assert ("gemm_fi_small_kernel" in plan.describe()) == (cfg < 0)
            tiles = -(-M // 32) * -(-N // 32)               # one workgroup per trial: a wave per tile, few steps
            assert ("gemm_fi_trial_kernel" in plan.describe()) == (cfg < 0 and tiles <= 16 and tiles * (K // 16) <= 128)
            faults = _faults(plan.desc, n, seed=7 * n + policy, kinds="eprcx" if n > 5 else "eprc")
            if n <= 2:                                  # every kind comes up
                faults = np.concatenate([_faults(plan.desc, n, seed=n + policy, kinds=k) for k in "eprc"])
            out = []
            for at in range(0, len(faults), n):
                d_f, d_r = fi.to_device(faults[at:at + n]), fi.empty_results(n)
                d_c = torch.full((n, M, N), 7.0, device="cuda")
                plan.fi_gemm_inject_batch(d_f, n, policy, d_r, d_c)
                out += [fi.results_to_host(d_r).tobytes(), d_c.cpu().numpy().tobytes()]
                d_h = torch.full((n, M, N), 7, dtype=torch.int16, device="cuda")
                plan.fi_gemm_inject_batch_act(d_f, n, policy, d_r, d_h)
                out += [fi.results_to_host(d_r).tobytes(), d_h.cpu().numpy().tobytes()]
                plan.fi_gemm_inject_batch_noalloc(d_f, n, policy, d_r)
                out += [fi.results_to_host(d_r).tobytes()]
            got.append(out)
            plan.destroy()
        assert got[0] == got[1], [i for i, (a, b) in enumerate(zip(*got)) if a != b]


@pytest.mark.parametrize("shape", [(1, 1, 16, 16), (33, 140, 80, 16), (64, 128, 128, 64), (65, 31, 576, 64)])
@pytest.mark.parametrize("n", [1, 3, 9])
@pytest.mark.parametrize("fmt", [orc.FP16, orc.BF16])
def test_small_next_layer_batches_equal_the_large_kernels(shape, n, fmt):
    # every trial its own A operand: equal to the plan's, a few words changed, Inf and NaN among them
    import torch
    M, N, K, kb = shape
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=M * N + K)
    rng = np.random.default_rng(n + K)
    stack = np.repeat(Aw[None], n, axis=0)
    for t in range(1, n):
        for _ in range(t):
            stack[t, rng.integers(M), rng.integers(K)] ^= np.uint16(1 << rng.integers(16))
    if n > 3:
        stack[3, M - 1, K - 1] = 0x7FFF                 # NaN in both formats
        stack[4, 0, 0] = 0x7F80 if fmt == orc.BF16 else 0x7C00
    d_A, d_B, d_s = fi.words_to_device(Aw), fi.words_to_device(Bw), fi.words_to_device(stack)
    for policy, bound in ((wl.CORRECT_ZERO, fi.BOUND_ROWCOL), (wl.CORRECT_RECOMPUTE, fi.BOUND_GLOBAL), (wl.CORRECT_NONE, fi.BOUND_EXPONENT)):
        got = []
        for cfg in (-1, 1, 2):                          # a wave per tile; persistent (K % 64 == 0); one workgroup per tile
            plan = fi.Plan(fi.plan_desc(M, N, K, kb, fmt, bound_mode=bound), d_A, d_B)
            plan.tune(cfg)
            d_r = fi.empty_results(n)
            d_c = torch.full((n, M, N), 7.0, device="cuda")
            plan.fi_gemm_propagate_batch(d_s, M * K, n, policy, d_r, d_c)
            recs = fi.results_to_host(d_r)
            plan.fi_gemm_propagate_batch(d_s, 0, n, policy, d_r)          # everybody the plan's own operand
            got.append((recs.tobytes(), d_c.cpu().numpy().view(np.uint32), fi.results_to_host(d_r).tobytes()))
            plan.destroy()
        assert not any(got[0][2][q] for q in range(len(got[0][2]))) or bound == fi.BOUND_EXPONENT
        for other in got[1:]:
            assert got[0][0] == other[0] and got[0][2] == other[2]
            assert np.array_equal(got[0][1], other[1])        # NaN words too
