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


def _side(M, N, K, n, cus):
    """Which kernel a next-layer batch without outputs goes to while no tile configuration is chosen."""
    up = lambda v, d: -(-v // d)
    steps = n * up(M, 32) * up(N, 128) * 4 * (K // 16) / (4.0 * cus)
    rounds, theirs = n * up(M, 32) * up(N, 128) / (2.0 * cus), n * up(M, 128) * up(N, 128) / (2.0 * cus)
    line = 0.8 + theirs if K >= 640 else 0.8 + 1.25 * theirs if K >= 384 and theirs <= 1 else 1.0 + 2.0 * theirs
    if steps <= 160 and rounds <= line:
        return "small"
    wide = up(n * (M // 256) * (N // 256), cus) if K >= 3072 and M % 256 == 0 and N % 256 == 0 else 0
    return "256" if wide >= 2 and 10 * n * (M // 256) * (N // 256) >= 9 * wide * cus else "128"


# n for 256 CUs, either side of each line: the first of K = 640 and of K = 384, that one's end where the persistent
# kernel takes a second round; two rounds of 256 x 256 tiles, nine tenths full and just less, one round
@pytest.mark.parametrize("M,N,K,n,side", [
    (300, 200, 640, 29, "small"), (300, 200, 640, 30, "128"), (300, 200, 384, 32, "small"), (300, 200, 384, 33, "128"),
    (300, 200, 320, 50, "small"), (57, 61, 384, 521, "small"), (57, 61, 640, 521, "128"),
    (256, 256, 3072, 461, "256"), (256, 256, 3072, 460, "128"), (256, 256, 3072, 256, "128"), (512, 256, 4096, 256, "256"),
    (256, 256, 3008, 512, "128"), (260, 256, 3072, 300, "128")])
def test_next_layer_batches_either_side_of_the_lines_between_the_kernels(M, N, K, n, side):
    import torch
    assert _side(M, N, K, n, torch.cuda.get_device_properties(0).multi_processor_count) == side
    g = torch.Generator(device="cuda").manual_seed(n)
    a, b = torch.randn(M, K, generator=g, device="cuda").bfloat16(), torch.randn(N, K, generator=g, device="cuda").bfloat16()
    stack = a.expand(n, M, K).clone()
    for t in range(0, n, 4):                            # a row, every row, a row that is flagged; every fourth trial untouched
        stack[t, t % M] = stack[t, (t + 1) % M]
        if t + 2 < n:
            stack[t + 1, :, t % K] *= 2
            stack[t + 2, (t + 5) % M, t % K] = float("inf")
    got = []
    for cfg in (-1, 2):                                 # the library's choice; one workgroup per tile
        plan = fi.Plan(fi.plan_desc(M, N, K, 32, fi.BF16), a, b)
        plan.tune(cfg)
        d_r = fi.empty_results(n)
        plan.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_RECOMPUTE, d_r)
        got.append(fi.results_to_host(d_r))
        plan.destroy()
    assert got[0].tobytes() == got[1].tobytes(), [t for t in range(n) if got[0][t] != got[1][t]][:5]
    assert not got[0]["n_bitdiff"][3::4].any() and (got[0]["n_bitdiff"][1::4][:n // 4 - 1] > M * N // 2).all()
    assert (got[0]["n_flagged"][2::4] == N).all()


# Two or three rounds of 256 x 256 tiles on 256 CUs, either side of the lines in K, trials and padding; ragged tiles, which
# pad no more than the 128 x 128 shape's, and an odd number of k-tiles
@pytest.mark.parametrize("M,N,K,n", [(256, 256, 1536, 768), (256, 256, 1536, 690), (256, 256, 1408, 768), (250, 248, 2560, 512),
                                     (250, 248, 2560, 460), (500, 760, 1536, 128), (250, 390, 2560, 256), (256, 256, 1600, 768)])
def test_next_layer_batches_either_side_of_the_lines_between_the_tile_shapes(M, N, K, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    a, b = torch.randn(M, K, generator=g, device="cuda").bfloat16(), torch.randn(N, K, generator=g, device="cuda").bfloat16()
    stack = a.expand(n, M, K).clone()
    t = torch.arange(0, n, 3, device="cuda")
    stack[t, t * 7 % M, t * 13 % K] *= 3
    stack[t[::5], t[::5] * 5 % M, 0] = float("inf")
    got = []
    for cfg in (-1, 0, 1):
        plan = fi.Plan(fi.plan_desc(M, N, K, 32, fi.BF16), a, b)
        plan.tune(cfg)
        d_r = fi.empty_results(n)
        plan.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_RECOMPUTE, d_r)
        got.append(fi.results_to_host(d_r))
        plan.destroy()
    assert got[0].tobytes() == got[1].tobytes() == got[2].tobytes()
    assert (got[0]["n_bitdiff"][::3] > 0).all() and not got[0]["n_bitdiff"][1::3].any()


# Campaigns and next layers of the small kernels on dirty records: cleared inside the kernel on a plan's first stream and up to
# 512 trials, by a launch in front on a second stream, beyond, without allocations and under capture.
@pytest.mark.parametrize("n", [1, 3, 70, 512, 513])
def test_small_batches_write_whole_records(n):
    import torch
    M, N, K, fmt = 200, 130, 96, orc.FP16
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=n)
    one, plan = gu.make_plan(Aw, Bw, 32, fmt, cfg=2), gu.make_plan(Aw, Bw, 32, fmt)
    faults = fi.fi_sample_faults(1, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    faults[2::5] = fi.fi_sample_faults(2, 0, n, plan.desc, fi.KIND_ALL_B, 2)[2::5]
    faults[3::5] = fi.fi_sample_faults(3, 0, n, plan.desc, fi.KIND_ALL_PRODUCT, 4)[3::5]
    faults["row"][4::9] = 10 ** 7
    faults["kind"][6::9] = fi.SITE_NONE
    want = gu.gpu_campaign(one, faults, wl.CORRECT_ZERO).tobytes()
    d_f = fi.to_device(faults)
    stack = fi.words_to_device(Aw).expand(n, M, K).clone()
    stack[::2, 5] += 3
    d_r = fi.empty_results(n)
    one.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_ZERO, d_r)
    want_next = fi.results_to_host(d_r).tobytes()
    side = torch.cuda.Stream()

    def both(stream, call=plan.fi_gemm_inject_batch):
        a, b = fi.empty_results(n).fill_(0xFF), fi.empty_results(n).fill_(0xFF)
        torch.cuda.synchronize()
        call(d_f, n, wl.CORRECT_ZERO, a, stream=stream)
        plan.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_ZERO, b, stream=stream)
        return a, b

    def check(a, b, what):
        assert fi.results_to_host(a).tobytes() == want, what
        assert fi.results_to_host(b).tobytes() == want_next, what
    for rep in range(3):
        check(*both(None), ("first stream", rep))
        check(*both(side), ("second stream", rep))
        check(*both(None, plan.fi_gemm_inject_batch_noalloc), ("no allocations", rep))
    g = torch.cuda.CUDAGraph()
    plan.reserve(n, side)
    a, b = fi.empty_results(n), fi.empty_results(n)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            s = torch.cuda.current_stream().cuda_stream
            plan.fi_gemm_inject_batch(d_f, n, wl.CORRECT_ZERO, a, stream=s)
            plan.fi_gemm_propagate_batch(stack, M * K, n, wl.CORRECT_ZERO, b, stream=s)
    for rep in range(2):
        a.fill_(0xFF); b.fill_(0xFF)
        check(*both(None), ("between replays", rep))
        g.replay()
        torch.cuda.synchronize()
        check(a, b, ("replay", rep))
    one.destroy()
    plan.destroy()


# The handle of the streams of all host threads (hipStreamPerThread): calls on it, one after the other on the host, may run
# at the same time, and so share nothing that the plan keeps for a stream.
def test_one_handle_for_the_streams_of_all_threads():
    import threading
    import torch
    PER_THREAD = 2
    M, N, K, fmt, n, reps = 1100, 130, 96, orc.FP16, 24, 40
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=9)
    plan = gu.make_plan(Aw, Bw, 32, fmt)
    faults = [fi.fi_sample_faults(t + 1, 0, n, plan.desc, kind, 1) for t, kind in enumerate((fi.KIND_ALL_ACC, fi.KIND_ALL_B))]
    want = [gu.gpu_campaign(plan, f, wl.CORRECT_ZERO).tobytes() for f in faults]
    plan.destroy()
    plan = gu.make_plan(Aw, Bw, 32, fmt)                   # its first stream is the one below
    plan.reserve(n, PER_THREAD)
    d_f = [fi.to_device(f) for f in faults]
    out = [[fi.empty_results(n).fill_(0xFF) for _ in range(2 * reps)] for _ in range(2)]
    torch.cuda.synchronize()
    lock = threading.Lock()

    def calls(t):
        torch.cuda.set_device(0)
        for rep in range(reps):
            with lock:
                plan.fi_gemm_inject_batch(d_f[t], n, wl.CORRECT_ZERO, out[t][2 * rep], stream=PER_THREAD)
                plan.fi_gemm_inject_batch_affected(d_f[t], n, wl.CORRECT_ZERO, out[t][2 * rep + 1], stream=PER_THREAD)
    threads = [threading.Thread(target=calls, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t in range(2):
        for i, r in enumerate(out[t]):
            assert fi.results_to_host(r).tobytes() == want[t], (t, i)
    plan.destroy()
