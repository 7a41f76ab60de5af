"""GPU tests of what include/fi.h promises about plans: handles, streams, scratch, the default
slack for long K and the guard of the affected-tiles-only campaign."""
import ctypes as C

import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def test_a_destroyed_plan_is_refused_not_read():
    Aw, Bw = wl.gaussian(64, 64, 64, orc.BF16, seed=1)
    plan = gu.make_plan(Aw, Bw, 32, orc.BF16)
    h = C.c_void_p(plan.handle.value)
    plan.destroy()
    L = fi.lib()
    assert L.fi_plan_destroy(h) == fi.STATE
    out = C.c_void_p()
    assert L.fi_plan_buffer(h, 0, C.byref(out)) == fi.STATE
    assert L.fi_plan_reserve(h, 8, None) == fi.STATE


def test_batches_of_one_plan_in_flight_on_two_streams_do_not_share_scratch():
    import torch
    w = wl.detector_stress()
    plan = gu.make_plan(w.A, w.B, w.kb, w.fmt)
    n = 2048
    fa = fi.fi_sample_faults(1, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    fb = fi.fi_sample_faults(2, 0, n, plan.desc, fi.KIND_ALL_B, 2)
    d_fa, d_fb = fi.to_device(fa), fi.to_device(fb)
    want_a = gu.gpu_campaign(plan, fa, wl.CORRECT_ZERO)
    want_b = gu.gpu_campaign(plan, fb, wl.CORRECT_ZERO)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    plan.reserve(n, s1)
    plan.reserve(n, s2)
    r_a, r_b = fi.empty_results(n), fi.empty_results(n)
    torch.cuda.synchronize()
    for _ in range(3):
        # each batch runs for milliseconds: the second is enqueued while the first is running
        plan.fi_gemm_inject_batch(d_fa, n, wl.CORRECT_ZERO, r_a, stream=s1)
        plan.fi_gemm_inject_batch(d_fb, n, wl.CORRECT_ZERO, r_b, stream=s2)
        torch.cuda.synchronize()
        assert fi.results_to_host(r_a).tobytes() == want_a.tobytes()
        assert fi.results_to_host(r_b).tobytes() == want_b.tobytes()
    plan.destroy()


def test_the_largest_next_layer_batch_does_not_depend_on_the_tiles_that_serve_it():
    # 256 x 256 x 3072: four tiles of the plan's 128 x 128 shape, one of the 256 x 256 shape that long-K batches take
    import torch
    n = 1 << 29
    a = torch.zeros((256, 3072), dtype=torch.float16, device="cuda")
    plan = fi.Plan(fi.plan_desc(256, 256, 3072, 32, fi.FP16), a, a)
    d_r = fi.empty_results(n)                                # 26 GB: refused before anything is enqueued
    with pytest.raises(fi.FiError, match="2\\^31 workgroups") as e:
        plan.fi_gemm_propagate_batch(a, 0, n, wl.CORRECT_ZERO, d_r)
    assert e.value.status == fi.UNSUPPORTED
    plan.destroy()
    del d_r
    torch.cuda.empty_cache()


# cfg None: the smallest batches' own kernels; 6: record fill, partition and two multi-trial launches.  3000
# trials are more than the scratch inside the plan holds: without the reserve the capture would allocate
@pytest.mark.parametrize("cfg,n", [(None, 200), (6, 200), (6, 3000)])
def test_reserve_then_capture_without_an_eager_call_first(cfg, n):
    import torch
    w = wl.tiny()
    plan = gu.make_plan(w.A, w.B, w.kb, w.fmt, cfg=cfg)
    assert ("gemm_fi_small_kernel" in plan.describe()) == (cfg is None)
    faults = fi.fi_sample_faults(9, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    d_f, d_r = fi.to_device(faults), fi.empty_results(n)
    side = torch.cuda.Stream()
    plan.reserve(n, side)                      # no batch has run on `side` yet
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_ZERO, d_r, stream=torch.cuda.current_stream().cuda_stream)
    want = gu.gpu_campaign(plan, faults, fi.CORRECT_ZERO)
    for rep in range(3):
        d_r.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert fi.results_to_host(d_r).tobytes() == want.tobytes(), rep
    plan.destroy()


@pytest.mark.parametrize("fused", [False, True])
def test_a_batch_no_larger_than_any_before_allocates_nothing_whatever_configuration_was_chosen_since(fused):
    # warm up with the batch, choose a tile configuration, capture the same batch: an allocation
    # inside the capture would be an error.  200 trials fit the plan's own scratch, 3000 do not.
    import torch
    w = wl.tiny()
    for n in (200, 3000):
        plan = gu.make_plan(w.A, w.B, w.kb, w.fmt)
        faults = fi.fi_sample_faults(9, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
        d_f, d_r = fi.to_device(faults), fi.empty_results(n)
        d_h = torch.empty((n, w.M, w.N), dtype=torch.int16, device="cuda") if fused else None

        def call(stream=None):
            if fused:
                plan.fi_gemm_inject_batch_act(d_f, n, fi.CORRECT_ZERO, d_r, d_h, stream=stream)
            else:
                plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_ZERO, d_r, stream=stream)
        sides = [torch.cuda.Stream(), torch.cuda.Stream()]
        for side in sides:
            torch.cuda.synchronize()                               # both write the same records
            call(side)
        torch.cuda.synchronize()
        want, want_h = fi.results_to_host(d_r).tobytes(), d_h.clone() if fused else None
        plan.tune(6)
        for side in sides:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                with torch.cuda.graph(g, stream=side):
                    call(torch.cuda.current_stream().cuda_stream)
            for rep in range(3):
                d_r.zero_()
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                assert fi.results_to_host(d_r).tobytes() == want, (n, rep)
                assert not fused or torch.equal(d_h, want_h)
        plan.destroy()


def test_a_plan_of_few_rows_takes_little_more_than_its_padded_result():
    # C* is padded to 512 rows; nothing else of the plan is
    import torch
    M, N, K = 1, 1 << 18, 16
    Aw, Bw = wl.small_integers(M, N, K, orc.BF16, seed=1, lim=2, step=1)
    d_A, d_B = fi.words_to_device(Aw), fi.words_to_device(Bw)
    gu.make_plan(Aw, Bw[:64], 16, orc.BF16).destroy()              # the library's own state is there
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan = fi.Plan(fi.plan_desc(M, N, K, 16, orc.BF16), d_A, d_B)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    assert used < 1.1 * 512 * N * 4, used
    # and the affected-only campaign reads no more of the sums than there is
    faults = orc.make_faults([(orc.SITE_A, 0, 3, 0, 0x8000), (orc.SITE_B, 2, N - 1, 0, 0x8000), (orc.SITE_ACC, 0, N - 1, 0, 1 << 30)])
    d_r = fi.empty_results(3)
    plan.fi_gemm_inject_batch_affected(fi.to_device(faults), 3, wl.CORRECT_ZERO, d_r)
    assert fi.results_to_host(d_r).tobytes() == gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO).tobytes()
    plan.destroy()


@pytest.mark.parametrize("cfg", [0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("fmt", [orc.FP16, orc.BF16])
def test_rows_of_all_maximal_same_sign_products_are_never_flagged(cfg, fmt):
    # The worst case for "a clean element is not flagged": every product of a row equals
    # ra_i * cb_j with one sign, so the exact sum IS K * ra_i * cb_j and only the slack factor
    # separates it from the bound.  K = 4096 with the default slack, every tile shape.
    M, N, K, kb = 160, 136, 4096, 64
    rng = np.random.default_rng(cfg)
    mant = rng.integers(128, 256, size=M) / 128.0            # 8 significant bits: exact in both formats
    a = np.repeat(mant[:, None], K, axis=1).astype(np.float32)
    a[::3] *= -1
    b = np.repeat((rng.integers(128, 256, size=N) / 128.0)[:, None], K, axis=1).astype(np.float32)
    Aw, Bw = wl.to_words(a, fmt), wl.to_words(b, fmt)
    plan = gu.make_plan(Aw, Bw, kb, fmt, cfg=cfg)
    faults = orc.make_faults([(orc.SITE_NONE, 0, 0, 0, 0)] * 3)
    recs = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    assert not recs["n_flagged"].any() and not recs["n_bitdiff"].any() and not recs["n_dev_pre"].any()
    # and the fault-free result sits right under the bound (so the test has teeth)
    cs = np.abs(plan.buffer_to_host(fi.BUF_C_STAR))
    T = np.float32(K) * np.abs(a[:, :1]) * np.abs(b[:, 0])[None, :]
    assert np.all(cs <= T * np.float32(1 + 2.0 ** -11)) and np.all(cs >= T * np.float32(1 - 2.0 ** -11))
    plan.destroy()


def _edge_operands(edge, M, N, K):
    A, B = np.ones((M, K), np.float32), np.full((N, K), 0.5, np.float32)
    if edge == "zero":                                  # thresholds of 0
        A[3] = A[M - 1] = 0
        B[5] = B[N - 1] = 0
    elif edge == "infinite":                            # row factors of Inf, of a column of zeros a NaN: flagged
        A[:] = 1e-3
        A[2] = A[M - 1] = 3.3e38
        B[:] = 1e-30
        B[7] = 0
    return wl.to_words(A, orc.BF16), wl.to_words(B, orc.BF16)


# Every element equal to its threshold; rows and columns of zeros; thresholds that are Inf and NaN.  Whole tiles and
# ragged ones, whose elements beyond the problem have no threshold.
@pytest.mark.parametrize("edge", ["equal", "zero", "infinite"])
@pytest.mark.parametrize("M,N", [(128, 128), (70, 100)])
@pytest.mark.parametrize("cfg", [0, 1, 3, 4, 5, 6, None])
def test_flags_at_the_edges_of_the_thresholds_equal_the_one_trial_kernels(edge, M, N, cfg):
    import torch
    K, n = 128, 700 if cfg is None else 41              # None: the shape that many trials get by themselves
    Aw, Bw = _edge_operands(edge, M, N, K)
    faults = np.zeros(n, fi.FAULT_DTYPE)
    rng = np.random.default_rng(M)
    faults["kind"] = fi.SITE_ACC
    faults["row"] = rng.choice([0, 2, 3, M - 1], n)
    faults["col"] = rng.choice([1, 5, 7, N - 1], n)
    faults["kblock"] = K // 32 - 1
    faults["xor_mask"] = 1 << rng.integers(0, 32, n)
    faults["kind"][::9] = fi.SITE_NONE
    got = []
    for c in (2, cfg):
        plan = gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=c, gamma=1.0)
        recs, out = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO, want_c=True)
        got.append((gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO).tobytes(), recs.tobytes(), out.tobytes()))
        if c in (0, 1, 2, None):                        # the next layer: flagged and unchanged, flagged and changed
            stack = fi.words_to_device(Aw).expand(3, M, K).clone()
            stack[1] += 1
            d_r = fi.empty_results(3)
            plan.fi_gemm_propagate_batch(stack, M * K, 3, wl.CORRECT_ZERO, d_r)
            got[-1] += (fi.results_to_host(d_r).tobytes(),)
        plan.destroy()
    assert got[0][:3] == got[1][:3]
    assert len(got[1]) == 3 or got[0][3] == got[1][3]
    flagged = np.frombuffer(got[0][1], recs.dtype)["n_flagged"]
    clean = {"equal": 0, "zero": 0, "infinite": 2}[edge]
    assert (flagged[::9] == clean).all() and flagged.max() > clean


def test_default_slack_for_long_K_matches_the_oracle_and_keeps_clean_trials_masked():
    M, N, K, kb, fmt = 40, 72, 8192, 64, orc.BF16
    a = np.full((M, K), 143.0 / 128.0, np.float32)           # sums that round upwards step after step
    b = np.full((N, K), 143.0 / 128.0, np.float32)
    a[5:9] = np.random.default_rng(0).standard_normal((4, K)).astype(np.float32)
    Aw, Bw = wl.to_words(a, fmt), wl.to_words(b, fmt)
    plan = gu.make_plan(Aw, Bw, kb, fmt)
    p = orc.problem(M, N, K, kb, fmt)
    assert p.gamma == np.float32(1 + 2.0 ** -10)
    faults = fi.fi_sample_faults(3, 0, 64, plan.desc, fi.KIND_ALL_ACC, 1)
    faults[:4]["kind"] = 0
    recs = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    ora = orc.campaign(p, Aw, Bw, gu.to_orc_faults(faults), wl.CORRECT_ZERO, orc.MODE_AFFECTED)
    assert not recs["n_flagged"][:4].any()
    ra, cb, _ = orc.rowcol_absmax(p, Aw, Bw)
    s = gu.compare_records(recs, ora, faults, site_tol=2.0 ** -12 * K * float(ra.max()) * float(cb.max()))
    assert not s["mismatches"], s["mismatches"][:5]
    plan.destroy()


def test_affected_only_campaign_refuses_a_plan_whose_clean_result_is_flagged():
    # Under the exponent-only bound any |C*| >= 2^17 is flagged in every trial of a full campaign;
    # the affected-tiles-only campaign would never visit it, so it must refuse.
    M, N, K, kb, fmt = 64, 64, 64, 32, orc.BF16
    Aw, Bw = wl.small_integers(M, N, K, fmt, seed=3, lim=2, step=1)
    big = wl.to_words(np.full(K, 64.0, np.float32), fmt)
    Aw = Aw.copy(); Bw = Bw.copy()
    Aw[7, :] = big; Bw[9, :] = big                           # C*[7, 9] = 64 * 64 * 64 = 2^18
    plan = gu.make_plan(Aw, Bw, kb, fmt, bound_mode=fi.BOUND_EXPONENT)
    p = orc.problem(M, N, K, kb, fmt, bound_mode=orc.BOUND_EXPONENT)
    faults = orc.make_faults([(orc.SITE_NONE, 0, 0, 0, 0), (orc.SITE_ACC, 1, 1, 0, 1 << 22),
                              (orc.SITE_ACC, 7, 9, 1, 1 << 31)])
    recs = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO)
    for t in range(len(faults)):
        o = orc.trial(p, Aw, Bw, faults[t:t + 1], wl.CORRECT_ZERO, orc.MODE_FULL)
        assert int(recs["n_flagged"][t]) == int(o["n_flagged"]) >= 1, t
    d_r = fi.empty_results(len(faults))
    with pytest.raises(fi.FiError) as e:
        plan.fi_gemm_inject_batch_affected(fi.to_device(faults), len(faults), wl.CORRECT_ZERO, d_r)
    assert e.value.status == fi.UNSUPPORTED
    plan.destroy()
    # the same operands under the operand-derived bound: nothing clean is flagged, the call works
    plan = gu.make_plan(Aw, Bw, kb, fmt)
    plan.fi_gemm_inject_batch_affected(fi.to_device(faults), len(faults), wl.CORRECT_ZERO, d_r)
    assert fi.results_to_host(d_r).tobytes() == gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO).tobytes()
    plan.destroy()


def test_operands_ending_at_the_end_of_their_allocation_short_K():
    # K = 16 and 48 with packed rows: the one-trial kernel's k-tile is 64 wide, so chunks past K
    # must be fetched from inside the row.  The operands sit at the very end of their buffers.
    import torch
    fmt = orc.BF16
    for (M, N, K, kb) in [(128, 128, 16, 16), (130, 70, 48, 16)]:
        Aw, Bw = wl.small_integers(M, N, K, fmt, seed=K, lim=2, step=1)
        pool_a = torch.zeros(M * K + 4096, dtype=torch.int16, device="cuda")
        pool_b = torch.zeros(N * K + 4096, dtype=torch.int16, device="cuda")
        d_A = pool_a[4096:].view(M, K); d_B = pool_b[4096:].view(N, K)
        d_A.copy_(fi.words_to_device(Aw)); d_B.copy_(fi.words_to_device(Bw))
        plan = fi.Plan(fi.plan_desc(M, N, K, kb, fmt), d_A, d_B)
        p = orc.problem(M, N, K, kb, fmt)
        assert np.array_equal(plan.buffer_to_host(fi.BUF_C_STAR).view(np.uint32), orc.gemm(p, Aw, Bw).view(np.uint32))
        faults = orc.make_faults([(orc.SITE_ACC, M - 1, N - 1, K // kb - 1, 1 << 30), (orc.SITE_A, M - 1, K - 1, 0, 0x8000),
                                  (orc.SITE_B, K - 1, N - 1, 0, 0x8000), (orc.SITE_PRODUCT, 1, 2, K - 1, 0x4000)])
        recs = gu.gpu_campaign(plan, faults, wl.CORRECT_RECOMPUTE)
        ora = orc.campaign(p, Aw, Bw, faults, wl.CORRECT_RECOMPUTE, orc.MODE_AFFECTED)
        s = gu.compare_records(recs, ora, faults, exact_words=True)
        assert not s["mismatches"], s["mismatches"]
        plan.destroy()


# A graph holds the scratch of its batch: a later reserve for as many trials or fewer leaves it, and gives the affected-only
# campaign its room elsewhere (1152 columns: nine tiles of 128, from eight on it has a use for it).
@pytest.mark.parametrize("n,first", [(100, False), (2000, False), (2000, True)])
def test_a_reserve_after_the_capture_leaves_what_the_graph_holds(n, first):
    import torch
    Aw, Bw = wl.gaussian(130, 1152, 128, orc.BF16, seed=n)
    plan = gu.make_plan(Aw, Bw, 32, orc.BF16, cfg=6)
    faults = fi.fi_sample_faults(9, 0, n, plan.desc, fi.KIND_MIX_ACC_A, 1)
    d_f, d_r, d_a = fi.to_device(faults), fi.empty_results(n), fi.empty_results(n)
    side = torch.cuda.Stream()
    if not first:
        plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_ZERO, d_r)
        torch.cuda.synchronize()
    plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_ZERO, d_r, stream=side)
    torch.cuda.synchronize()
    want = fi.results_to_host(d_r).tobytes()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            plan.fi_gemm_inject_batch(d_f, n, fi.CORRECT_ZERO, d_r, stream=torch.cuda.current_stream().cuda_stream)
    plan.reserve(n // 2, side)
    plan.reserve(n, side)
    for rep in range(3):
        other = [torch.full((1 << k,), -1, dtype=torch.int32, device="cuda") for k in range(10, 20)]   # of the sizes of such scratch
        d_r.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert fi.results_to_host(d_r).tobytes() == want, rep
        assert all(bool((x == -1).all()) for x in other), rep
        plan.fi_gemm_inject_batch_affected(d_f, n, fi.CORRECT_ZERO, d_a, stream=side)
        torch.cuda.synchronize()
        assert fi.results_to_host(d_a).tobytes() == want, rep
    plan.destroy()
