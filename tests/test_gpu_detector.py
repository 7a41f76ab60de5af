"""The standalone detector / corrector at the sizes where its walk over the flat outputs can go wrong:
narrow and odd rows, vectors that span rows and trials, unaligned buffers, several rounds of its
grid.  Against the definition, element by element, in binary32 (the threshold's three roundings)."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,batch,shift", [
    (1, 1, 1, 0), (1, 1, 9000, 0), (3, 2, 700, 0), (5, 3, 401, 0),     # N < 4: element by element
    (1, 5, 1000, 0), (7, 5, 333, 0), (33, 7, 70, 0),                   # vectors over rows and trials
    (100, 64, 17, 0), (2, 4, 2049, 0), (257, 1028, 3, 0),              # whole vectors in a row
    (100, 64, 17, 1), (33, 7, 70, 2), (3, 4099, 2, 3),                 # buffers off alignment
    (1000, 1003, 70, 0), (1000, 1004, 70, 0), (100, 7, 25000, 2),      # more chunks than workgroups
    (1, 1024, 3, 0), (3, 2052, 40, 0), (1000, 1028, 70, 0), (1, 1028, 65535, 0),   # waves that hand over together
])
@pytest.mark.parametrize("bound", [fi.BOUND_ROWCOL, fi.BOUND_GLOBAL])
def test_detector_equals_its_definition(M, N, batch, shift, bound):
    import torch
    Aw, Bw = wl.gaussian(M, N, 64, orc.BF16, seed=M + N)
    plan = gu.make_plan(Aw, Bw, 32, orc.BF16, bound_mode=bound)
    kra = torch.from_numpy(plan.buffer_to_host(fi.BUF_KRA)).cuda()
    cb = torch.from_numpy(plan.buffer_to_host(fi.BUF_CB)).cuda()
    cstar = torch.from_numpy(plan.buffer_to_host(fi.BUF_C_STAR)).cuda()
    gamma = np.float32(1 + 2.0 ** -11)
    T = (kra[:, None] * cb[None, :]) * float(gamma)
    if bound == fi.BOUND_GLOBAL:
        T = torch.full_like(T, float(np.float32(np.float32(kra.max().item()) * np.float32(cb.max().item())) * gamma))
    g = torch.Generator(device="cuda").manual_seed(M * 31 + N)
    n = batch * M * N
    src = T.expand(batch, M, N).reshape(-1) * (torch.rand(n, generator=g, device="cuda") * 1.0005)
    at = torch.randint(0, n, (max(1, n // 50),), generator=g, device="cuda")
    src[at] = torch.tensor([float("nan"), float("inf"), -3.0e38, 0.0], device="cuda")[torch.arange(len(at), device="cuda") % 4]
    src[torch.randint(0, n, (max(1, n // 9),), generator=g, device="cuda")] *= -1
    want = ~(src.view(batch, M, N).abs() <= T)
    for policy in (wl.CORRECT_NONE, wl.CORRECT_ZERO, wl.CORRECT_RECOMPUTE):
        c_buf = torch.full((n + 8,), 7.0, device="cuda")
        f_buf = torch.full((n + 8,), 9, dtype=torch.uint8, device="cuda")
        c, fl = c_buf[shift:shift + n], f_buf[shift:shift + n]
        c.copy_(src)
        cnt = torch.full((batch,), -1, dtype=torch.int32, device="cuda")
        plan.fi_detect_correct(c, batch, policy, fl, cnt)
        assert torch.equal(fl.view(batch, M, N) != 0, want)
        assert torch.equal(cnt, want.sum(dim=(1, 2), dtype=torch.int32))
        ref = src.view(batch, M, N)
        if policy != wl.CORRECT_NONE:
            ref = torch.where(want, cstar.expand(batch, M, N) if policy == wl.CORRECT_RECOMPUTE else torch.zeros((), device="cuda"), ref)
        assert torch.equal(c.view(torch.int32), ref.reshape(-1).view(torch.int32))
        assert bool((c_buf[:shift] == 7).all()) and bool((c_buf[shift + n:] == 7).all())     # nothing outside
        assert bool((f_buf[:shift] == 9).all()) and bool((f_buf[shift + n:] == 9).all())
    plan.destroy()


# Counters holding anything: cleared inside the kernel on a plan's first stream and up to 512 trials, by a launch in front
# on a second stream, beyond and under capture.  Long rows, whose waves hand over together, and short ones.
@pytest.mark.parametrize("batch,M,N", [(512, 3, 1028), (513, 3, 1028), (300, 40, 33), (1, 500, 700)])
def test_detector_clears_its_counters(batch, M, N):
    import torch
    plan = gu.make_plan(*wl.gaussian(M, N, 64, orc.BF16, seed=N), 32, orc.BF16)
    c = torch.zeros(batch, M, N, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(batch)
    hits = torch.rand(batch, M, N, generator=g, device="cuda") < torch.rand(batch, 1, 1, generator=g, device="cuda") ** 4
    c[hits] = float("inf")
    want = hits.sum(dim=(1, 2), dtype=torch.int32)
    cnt = torch.empty(batch, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()

    def check(stream, what):
        cnt.fill_(-7)
        torch.cuda.synchronize()
        plan.fi_detect_correct(c, batch, wl.CORRECT_NONE, None, cnt, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(cnt, want), what
    graph = torch.cuda.CUDAGraph()
    for rep in range(2):
        check(None, ("first stream", rep))
        check(side, ("second stream", rep))
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            plan.fi_detect_correct(c, batch, wl.CORRECT_NONE, None, cnt, stream=torch.cuda.current_stream().cuda_stream)
    for rep in range(2):
        cnt.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(cnt, want), ("replay", rep)
        check(None, ("between replays", rep))
    plan.destroy()


@pytest.mark.parametrize("cfg", [-1, 2, 3, 6])          # element by element; through the largest excess over T
def test_fused_detector_tells_subnormal_values_from_a_subnormal_threshold(cfg):
    # ra = cb = 2^-70, K = 128: T = 2^-133 * (1 + 2^-11) = 65568 units of 2^-149.  The fault writes its mask into an
    # accumulator of +0, whose value is then that many units: flagged from 65569 on.
    M, N, K = 64, 64, 128
    word = np.uint16((127 - 70) << 7)                    # BF16 2^-70
    A, B = np.zeros((M, K), np.uint16), np.zeros((N, K), np.uint16)
    A[:, 0], B[:, 1] = word, word                        # every product 0
    plan = fi.Plan(fi.plan_desc(M, N, K, 32, fi.BF16), fi.words_to_device(A), fi.words_to_device(B))
    plan.tune(cfg)
    masks = [1, 0x10000, 0x1001F, 0x10020, 0x10021, 0x10022, 0x80010020, 0x80010021, 0x20000, 0x7F800000, 0x7FC00000]
    faults = np.zeros(len(masks), fi.FAULT_DTYPE)
    faults["kind"], faults["row"], faults["col"], faults["kblock"] = fi.SITE_ACC, 5, 40, 3
    faults["xor_mask"] = masks
    d_r = fi.empty_results(len(masks))
    plan.fi_gemm_inject_batch(fi.to_device(faults), len(masks), fi.CORRECT_ZERO, d_r)
    r = fi.results_to_host(d_r)
    want = [int((m & 0x7FFFFFFF) > 0x10020) for m in masks]
    assert r["n_flagged"].tolist() == want and r["n_bitdiff"].tolist() == [1] * len(masks)
    plan.destroy()
