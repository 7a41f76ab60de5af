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


def _records(plan, faults):
    n = len(faults)
    d_f, d_r, d_a = fi.to_device(faults), fi.empty_results(n), fi.empty_results(n)
    plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_RECOMPUTE, d_r)
    plan.fi_gemm_inject_batch_affected(d_f, n, fi.CORRECT_RECOMPUTE, d_a)
    return fi.results_to_host(d_r).tobytes() + fi.results_to_host(d_a).tobytes()


def _make(M, N, K, seed, scale=1.0, b_layout=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = (torch.randn(M, K, generator=g, device="cuda") * scale).bfloat16()
    b = (torch.randn(N, K, generator=g, device="cuda") * scale).bfloat16()
    return fi.Plan(fi.plan_desc(M, N, K, 16, fi.BF16, b_layout=b_layout), a, b if b_layout == 0 else b.t().contiguous())


# Plans over memory that destroyed ones of other sizes and huge results have left; several threads, each with a
# stream of its own, whose plans take and give such memory at the same time.
def test_plans_over_the_memory_of_destroyed_ones():
    import threading
    import torch
    shapes = [(512, 1500, 208, 0), (300, 700, 64, 1), (1030, 900, 80, 0), (400, 1100, 128, 1)]
    kept = [_make(*s[:3], seed=k, b_layout=s[3]) for k, s in enumerate(shapes)]       # none has had another's memory
    faults = [np.concatenate([fi.fi_sample_faults(9, 0, 40, p.desc, k, 1) for k in (fi.KIND_MIX_ACC_A, fi.KIND_ALL_B, fi.KIND_ALL_PRODUCT)])
              for p in kept]
    want = [_records(p, f) for p, f in zip(kept, faults)]
    wrong = []

    def sweep(worker):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for rep in range(6):
                k = (worker + rep) % len(shapes)
                M, N, K, layout = shapes[k]
                _make(M, N, K, seed=50 + rep, scale=1e15, b_layout=layout).destroy()
                plan = _make(M, N, K, seed=k, b_layout=layout)
                if _records(plan, faults[k]) != want[k]:
                    wrong.append((worker, rep, k))
                plan.destroy()
    sweep(0)
    assert not wrong
    threads = [threading.Thread(target=sweep, args=(w,)) for w in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for p in kept:
        p.destroy()


def test_memory_of_destroyed_plans_is_bounded_and_given_back():
    import torch
    torch.cuda.synchronize()
    MB = 1 << 20
    before = torch.cuda.mem_get_info()[0]
    for m in range(12):                                     # 10 .. 130 MB each, never the same
        _make(1024 + 512 * m, 1024 + 256 * m, 16, seed=m).destroy()
        torch.cuda.empty_cache()
        assert before - torch.cuda.mem_get_info()[0] <= (256 + 32) * MB, m
    for m in range(20):                                     # small ones that have no use for it
        _make(64, 64, 16, seed=m).destroy()
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] <= 48 * MB


def test_memory_of_destroyed_plans_is_given_back_on_demand():
    import torch
    plan = _make(300, 700, 64, seed=1)
    faults = fi.fi_sample_faults(9, 0, 40, plan.desc, fi.KIND_MIX_ACC_A, 1)
    want = _records(plan, faults)
    fi.fi_release_memory()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    for m in range(3):
        _make(2048, 2048 + 1024 * m, 16, seed=m).destroy()             # 34 .. 67 MB
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] >= 64 << 20           # kept
    fi.fi_release_memory()
    assert before - torch.cuda.mem_get_info()[0] <= 8 << 20
    assert _records(plan, faults) == want                               # the live plan is as it was
    other = _make(300, 700, 64, seed=1)
    assert _records(other, faults) == want
    plan.destroy()
    other.destroy()


# A plan of another device than the current one: destroyed behind work that still reads it, its memory at once a new plan's.
@pytest.mark.parametrize("rep", range(3))
def test_plans_of_another_device_than_the_current_one(rep):
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("one GPU")
    with torch.cuda.device(1):
        other = _make(512, 1500, 208, seed=rep, scale=1e15)
        plan = _make(512, 1500, 208, seed=7)
        faults = fi.fi_sample_faults(9, 0, 2000, plan.desc, fi.KIND_MIX_ACC_A, 1)
        d_f, d_r, d_s = fi.to_device(faults), fi.empty_results(2000), fi.empty_results(2000)
        plan.fi_gemm_inject_batch(d_f, 2000, fi.CORRECT_ZERO, d_r)
        torch.cuda.synchronize()
        want = fi.results_to_host(d_r).tobytes()
        plan.fi_gemm_inject_batch(d_f, 2000, fi.CORRECT_ZERO, d_s)
    with torch.cuda.device(0):
        plan.destroy()
        assert torch.cuda.current_device() == 0
    with torch.cuda.device(1):
        _make(512, 1500, 208, seed=rep, scale=1e15).destroy()
        torch.cuda.synchronize()
        assert fi.results_to_host(d_s).tobytes() == want
        other.destroy()
