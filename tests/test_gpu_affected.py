"""The affected-only campaign's element and row / column kernels at the sizes where their indexing
can go wrong, against the full campaign: the records have to be the same bytes (every element is
accumulated by the same sequence of matrix steps)."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def _faults(desc, n, seed, kinds):
    parts = [fi.fi_sample_faults(seed + q, 0, n, desc, k, b)
             for q, (k, b) in enumerate(((fi.KIND_ALL_ACC, 1), (fi.KIND_ALL_PRODUCT, 4), (fi.KIND_ALL_A, 1), (fi.KIND_ALL_B, 2)))]
    rng = np.random.default_rng(seed)
    pick = rng.choice([q for q in range(4) if "eprc"[q] in kinds], size=n)
    f = np.stack(parts)[pick, np.arange(n)]
    if "x" in kinds:                                    # no fault, and sites outside the problem
        f["kind"][rng.integers(0, n, n // 8 + 1)] = fi.SITE_NONE
        f["row"][rng.integers(0, n, n // 8 + 1)] = 10 ** 7
        f["kind"][rng.integers(0, n, n // 16 + 1)] = 77
    return f


# (M, N, K, k-block), trials, kinds (e element, p product, r A rows, c B columns, x none / invalid)
@pytest.mark.parametrize("shape,n,kinds", [
    ((1, 1, 16, 16), 3, "eprcx"),            # one step, one element; fewer trials than a wave takes
    ((5, 3, 48, 16), 70, "eprc"),            # K below a k-tile
    ((130, 70, 528, 16), 513, "eprcx"),      # one trial beyond a chunk; K past one 512-wide piece, ragged k-tile
    ((257, 131, 1040, 16), 1100, "eprcx"),   # K past one 1024-wide piece; N not a multiple of 4
    ((300, 515, 192, 32), 640, "r"),         # A rows only: ten items in two chunks
    ((515, 300, 192, 64), 577, "c"),         # B columns only, a ragged last item
    ((33, 200, 4096, 64), 2500, "ep"),       # several pieces, shallow buffering (more than two waves a CU)
    ((64, 72, 5120, 64), 90, "eprx"),        # more pieces than buffers
])
@pytest.mark.parametrize("fmt", [orc.FP16, orc.BF16])
def test_affected_records_equal_the_full_campaigns(shape, n, kinds, fmt):
    import torch
    M, N, K, kb = shape
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=M + K)
    wide = np.zeros((M, K + 24), np.uint16)             # rows longer than K, the gap full of NaN
    wide[:] = 0x7FFF
    wide[:, :K] = Aw
    for policy, b_layout, check in ((wl.CORRECT_ZERO, 0, fi.PCHECK_NONE), (wl.CORRECT_RECOMPUTE, 1, fi.PCHECK_RANGE_MAX),
                                    (wl.CORRECT_NONE, 0, fi.PCHECK_BOUND)):
        bound = (fi.BOUND_ROWCOL, fi.BOUND_GLOBAL, fi.BOUND_EXPONENT)[policy]
        B = Bw if b_layout == 0 else np.ascontiguousarray(Bw.T)
        plan = fi.Plan(fi.plan_desc(M, N, K, kb, fmt, b_layout=b_layout, bound_mode=bound, lda=K + 24),
                       fi.words_to_device(wide), fi.words_to_device(B))
        plan.set_product_check(check)
        faults = _faults(plan.desc, n, seed=n + policy, kinds=kinds)
        want = gu.gpu_campaign(plan, faults, policy)
        # records 4 bytes off an 8-byte boundary once: no alignment is promised beyond the words'
        off = 4 if policy == wl.CORRECT_RECOMPUTE else 0
        buf = torch.full((n * 48 + off,), 0xAB, dtype=torch.uint8, device="cuda")
        plan.fi_gemm_inject_batch_affected(fi.to_device(faults), n, policy, buf[off:])
        got = fi.results_to_host(buf[off:])
        assert got.tobytes() == want.tobytes(), [(t, faults[t], got[t], want[t]) for t in range(n) if got[t] != want[t]][:3]
        plan.destroy()


# Operand faults whose workgroups leave their counts in reserved scratch, to be added up: a slot per tile of 128 and one
# trial more than an item, a row that lies in one slot of many (the others leave nothing), more slots than lanes that
# add up in one go, several tiles per slot
@pytest.mark.parametrize("M,N,n,kinds", [(70, 1025, 65, "r"), (1025, 70, 65, "c"), (1100, 64, 300, "r"), (64, 2100, 130, "erc"),
                                         (40, 2200, 1500, "eprcx"), (3000, 40, 9000, "rc")])
def test_affected_records_added_up_from_reserved_scratch(M, N, n, kinds):
    import torch
    fmt = orc.BF16
    Aw, Bw = wl.gaussian(M, N, 64, fmt, seed=M)
    plan = gu.make_plan(Aw, Bw, 32, fmt)
    faults = _faults(plan.desc, n, seed=n, kinds=kinds)
    want = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    d_f = fi.to_device(faults)

    def call(m, stream=None):
        buf = torch.full((m * 48,), 0xAB, dtype=torch.uint8, device="cuda")
        plan.fi_gemm_inject_batch_affected(d_f, m, wl.CORRECT_ZERO, buf, stream=stream)
        return buf
    # nothing reserved; reserved; a smaller batch, whose slots hold the counts of the larger one; a batch beyond
    # what is reserved; captured, where the scratch is not used
    few = max(n // 3, 1)
    got = [fi.results_to_host(call(n))]
    plan.reserve(few)
    got += [fi.results_to_host(call(n)), fi.results_to_host(call(few))]
    plan.reserve(n)
    got += [fi.results_to_host(call(n)), fi.results_to_host(call(few)), fi.results_to_host(call(n))]
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    plan.reserve(n, side)
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            buf = call(n, torch.cuda.current_stream().cuda_stream)
    for _ in range(2):
        buf.fill_(0xFF)
        g.replay()
        torch.cuda.synchronize()
        got.append(fi.results_to_host(buf))
    for k, r in enumerate(got):
        assert r.tobytes() == want[:len(r)].tobytes(), (k, [(t, faults[t], r[t], want[t]) for t in range(len(r)) if r[t] != want[t]][:3])
    plan.destroy()


def test_affected_records_where_the_fault_free_result_spans_4_gib():
    # C* addressed with 64 bits (rows kernel), one 16-wide step
    M, N, K, kb, fmt = 65600, 16400, 16, 16, orc.BF16
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=9)
    plan = gu.make_plan(Aw, Bw, kb, fmt)
    n = 12
    faults = _faults(plan.desc, n, seed=4, kinds="eprc")
    faults["kind"][:4] = (fi.SITE_A, fi.SITE_B, fi.SITE_A, fi.SITE_B)
    faults["row"][:4], faults["col"][:4] = (M - 1, K - 1, 3, 0), (K - 1, N - 1, 7, 16395)
    want = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    d_r = fi.empty_results(n)
    plan.fi_gemm_inject_batch_affected(fi.to_device(faults), n, wl.CORRECT_ZERO, d_r)
    assert fi.results_to_host(d_r).tobytes() == want.tobytes()
    plan.destroy()


@pytest.mark.parametrize("K,a,b,gamma,kind,masks", [
    (64, 2.0 ** -57, 2.0 ** 58, 1e22, fi.SITE_A, (0xF000, 0x7000, 0x3000)),   # cb * gamma beyond binary32, kra * cb * gamma not
    (16, 1.7265625 * 2.0 ** -77, 1.7265625 * 2.0 ** -77, 300.0, fi.SITE_A, (0x0600, 0x0400, 0x0200)),   # kra * cb: 1.49 -> 1 unit of 2^-149
    (64, 2.0 ** 20, 2.0 ** 20, 1e20, fi.SITE_A, (0x4000, 0x0080)),
    (64, 2.0 ** 58, 2.0 ** -57, 1e22, fi.SITE_B, (0xF000, 0x7000, 0x3000)),
])
@pytest.mark.parametrize("bound", [fi.BOUND_ROWCOL, fi.BOUND_GLOBAL])
def test_affected_records_at_extreme_thresholds(K, a, b, gamma, kind, masks, bound):
    # thresholds whose factors leave the normal range on the way: the flags are those of the three
    # roundings fl(fl(kra * cb) * gamma), as in the full campaign
    M, N, fmt = 70, 200, orc.BF16
    Aw = wl.to_words(np.full((M, K), a, np.float32), fmt)
    Bw = wl.to_words(np.full((N, K), b, np.float32), fmt)
    plan = gu.make_plan(Aw, Bw, 16, fmt, bound_mode=bound, gamma=gamma)
    rows = [(kind, r, c, 0, m) for m in masks for r, c in ((0, 0), (K - 1, K // 2), (5, K - 1))]
    faults = orc.make_faults(rows)
    want = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    d_r = fi.empty_results(len(faults))
    plan.fi_gemm_inject_batch_affected(fi.to_device(faults), len(faults), wl.CORRECT_ZERO, d_r)
    got = fi.results_to_host(d_r)
    assert got.tobytes() == want.tobytes(), [(faults[t], got[t], want[t]) for t in range(len(faults)) if got[t] != want[t]][:3]
    if gamma == 1e22:
        assert (want["n_flagged"] > 0).any()
    plan.destroy()
