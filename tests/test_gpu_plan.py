"""What a plan computes when it is created - C*, the magnitude sums, the operand maxima, the elements
of C* that its own detector flags - on both sides of the line between its two fault-free passes, in the
exact-arithmetic regime (integer operands: any summation order gives the same words)."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,kb,b_layout", [
    (1, 1, 16, 16, 0), (33, 65, 80, 16, 1), (300, 203, 176, 16, 0), (64, 512, 1040, 16, 1),   # a wave per 32 x 32 tile
    (4100, 3100, 1040, 16, 0), (40000, 60, 1024, 64, 1),                                      # large tiles, run twice
])
@pytest.mark.parametrize("bound", [fi.BOUND_ROWCOL, fi.BOUND_GLOBAL, fi.BOUND_EXPONENT])
def test_plan_buffers_and_clean_flags(M, N, K, kb, b_layout, bound):
    import torch
    fmt = orc.BF16
    Aw, Bw = wl.small_integers(M, N, K, fmt, seed=M + K, lim=4, step=1)
    Aw, Bw = Aw.copy(), Bw.copy()
    big = wl.to_words(np.full(K, 64.0, np.float32), fmt)
    Aw[M // 2, :], Bw[N - 1, :] = big, big                 # |C*| = 4096 K there: over 2^17 beyond K = 32
    d_B = fi.words_to_device(Bw if b_layout == 0 else np.ascontiguousarray(Bw.T))
    plan = fi.Plan(fi.plan_desc(M, N, K, kb, fmt, b_layout=b_layout, bound_mode=bound), fi.words_to_device(Aw), d_B)
    a = torch.from_numpy(orc.decode_array(Aw, fmt)).cuda().double()
    b = torch.from_numpy(orc.decode_array(Bw, fmt)).cuda().double()
    want = a @ b.t()
    assert torch.equal(torch.from_numpy(plan.buffer_to_host(fi.BUF_C_STAR)).cuda().double(), want)
    assert torch.equal(torch.from_numpy(plan.buffer_to_host(fi.BUF_S_ABS)).cuda().double(), a.abs() @ b.abs().t())
    assert np.array_equal(plan.buffer_to_host(fi.BUF_KRA), (K * a.abs().amax(1)).float().cpu().numpy())
    assert np.array_equal(plan.buffer_to_host(fi.BUF_CB), b.abs().amax(1).float().cpu().numpy())
    flagged = int((want.abs() >= 2 ** 17).sum()) if bound == fi.BOUND_EXPONENT else 0
    assert (flagged > 0) == (bound == fi.BOUND_EXPONENT and K > 32)
    d_f, d_r = fi.to_device(orc.make_faults([(orc.SITE_NONE, 0, 0, 0, 0)])), fi.empty_results(1)
    if flagged:
        with pytest.raises(fi.FiError, match="flags %d element" % flagged):
            plan.fi_gemm_inject_batch_affected(d_f, 1, fi.CORRECT_ZERO, d_r)
    else:
        plan.fi_gemm_inject_batch_affected(d_f, 1, fi.CORRECT_ZERO, d_r)
    # the campaign's own fault-free trial is the plan's result bit for bit
    plan.fi_gemm_inject_batch(d_f, 1, fi.CORRECT_NONE, d_r)
    rec = fi.results_to_host(d_r)[0]
    assert int(rec["n_flagged"]) == flagged and int(rec["n_bitdiff"]) == 0
    plan.destroy()
