"""The host code of plans - scratch, memory of destroyed plans, devices - over a stand-in for the HIP runtime."""
import pytest

import host_double


# A graph holds the addresses of the scratch that its batch was captured with.  512 x 3072: 24 tiles of 128 along the longer
# side, so the affected-only campaign has a use for parts.
@pytest.mark.parametrize("stream,n", [("SIDE", 8), ("SIDE", 2000), ("None", 2000)])
def test_reserve_leaves_the_scratch_of_a_batch_no_smaller(stream, n):
    host_double.run("""
    stream, n = %s, %d
    plan = create(512, 3072, 768)
    L.fi_plan_tune(plan, 6, -1, None)
    inject(plan, 1, OTHER if stream else None)          # a plan's first stream has scratch inside the plan
    assert inject(plan, n, stream) == 0
    held = scratch_of_last_batch()
    for m in (n, max(1, n // 4), n - 1):
        assert reserve(plan, m, stream) == 0
        assert all(D.double_is_live(w) for w in held), m
    D.double_capacity(D.double_in_use())                # nor where there is no memory left
    assert reserve(plan, n, stream) == 0 and inject(plan, n, stream) == 0
    assert scratch_of_last_batch() == held
    """ % (stream, n))


# What only makes a call faster breaks no capture: a reserve no larger than a batch before allocated nothing before there
# were parts.
@pytest.mark.parametrize("captures", ["SIDE", "OTHER"])
def test_reserve_of_what_is_there_under_capture(captures):
    host_double.run("""
    plan = create(512, 3072, 768)
    inject(plan, 1, OTHER)
    assert inject(plan, 2000, SIDE) == 0
    D.double_capture(%s, 1)
    D.double_forget()
    assert reserve(plan, 2000, SIDE) == 0 and reserve(plan, 300, SIDE) == 0
    assert D.double_unsafe_calls() == 0
    assert affected(plan, 2000, SIDE) == 0
    assert parts_used() == %s                           # another stream's capture does not keep it from them
    """ % (captures, captures == "OTHER"))


def test_parts_come_with_a_reserve_after_the_batch():
    host_double.run("""
    plan = create(512, 3072, 768)
    inject(plan, 1, OTHER)
    assert inject(plan, 4096, SIDE) == 0 and affected(plan, 4096, SIDE) == 0
    assert not parts_used()
    blocks = D.double_blocks()
    for n in (8, 4096, 500, 4096):                      # the smaller parts go when the larger ones come
        assert reserve(plan, n, SIDE) == 0
        assert D.double_blocks() == blocks + 1
        D.double_forget()
        assert affected(plan, n, SIDE) == 0
        assert parts_used(), n
    L.fi_plan_destroy(plan)
    assert D.double_blocks() == 1                       # the plan's own memory, kept for the next
    """)


# A reservation's room for the affected-only campaign survives a larger plain batch, wherever it lies.
@pytest.mark.parametrize("first_stream", [True, False])
@pytest.mark.parametrize("order", ["reserve", "batch, reserve"])
def test_a_larger_batch_keeps_the_parts(first_stream, order):
    host_double.run("""
    plan = create(512, 3072, 768)
    stream = %s
    inject(plan, 1, OTHER if stream else None)
    if %s:
        assert inject(plan, 1000, stream) == 0
    assert reserve(plan, 1000, stream) == 0
    for n in (1500, 3000, 20000):
        assert inject(plan, n, stream) == 0
        for m in (1000, 7):
            D.double_forget()
            assert affected(plan, m, stream) == 0
            assert parts_used(), (n, m)
    assert reserve(plan, 20000, stream) == 0            # and the larger reservation's are there
    D.double_forget()
    assert affected(plan, 4096, stream) == 0
    assert parts_used()
    L.fi_plan_destroy(plan)
    assert D.double_blocks() == 1
    """ % ("None" if first_stream else "SIDE", order != "reserve"))


# Parts in an allocation of their own that happens to lie right behind the scratch are not taken for a part of it.
def test_parts_right_behind_the_scratch_are_given_back():
    host_double.run("""
    D.double_packed()
    plan = create(512, 3072, 768)
    inject(plan, 1, OTHER)
    assert inject(plan, 1000, SIDE) == 0 and reserve(plan, 1000, SIDE) == 0
    for n in (1500, 3000):
        assert inject(plan, n, SIDE) == 0
        D.double_forget()
        assert affected(plan, 1000, SIDE) == 0
        assert parts_used()
    L.fi_plan_destroy(plan)
    assert D.double_blocks() == 1
    """)


# No room for the parts: the batch has its scratch all the same.
def test_a_larger_batch_without_memory_for_the_parts():
    host_double.run("""
    plan = create(512, 3072, 768)
    inject(plan, 1, OTHER)
    assert reserve(plan, 1000, SIDE) == 0
    D.double_capacity(D.double_in_use())
    assert inject(plan, 5000, SIDE) == 0
    assert all(D.double_is_live(w) for w in scratch_of_last_batch())
    D.double_forget()
    assert affected(plan, 1000, SIDE) == 0 and not parts_used()
    """)


# Memory of destroyed plans that the library keeps is given back where a stream's scratch finds no other.
@pytest.mark.parametrize("call", ["reserve(plan, 100000, SIDE)", "inject(plan, 100000, SIDE)", "inject(plan, 100000, None)"])
def test_scratch_takes_the_memory_of_destroyed_plans(call):
    host_double.run("""
    plan, other = create(512, 3072, 768), create(2048, 2048, 64)
    assert L.fi_plan_destroy(other) == 0
    kept = D.double_in_use()
    D.double_capacity(kept + 4096)
    assert %s == 0, L.fi_last_error()
    assert D.double_in_use() < kept
    D.double_capacity(D.double_in_use() + 4096)
    assert inject(plan, 10000000, SIDE) == fi.OOM       # as before where there is none to give back
    """ % call)


# All that the library keeps beyond its plans can be given back, on every GPU, and the next plan starts anew.
def test_release_memory():
    host_double.run("""
    plan = create(300, 700, 64)
    L.fi_plan_destroy(create(512, 3072, 768))
    fi_device = C.c_int(1)
    D.hipSetDevice(fi_device)
    L.fi_plan_destroy(create(512, 3072, 768))
    D.hipSetDevice(0)
    assert D.double_blocks() == 3 and D.double_host_blocks() == 1
    fi.fi_release_memory()
    assert D.double_blocks() == 1 and D.double_host_blocks() == 0     # the live plan's
    assert inject(plan, 40, None) == 0
    for _ in range(3):
        L.fi_plan_destroy(create(512, 3072, 768))
    assert D.double_blocks() == 2
    L.fi_plan_destroy(plan)
    fi.fi_release_memory()
    fi.fi_release_memory()
    assert D.double_blocks() == 0 and D.double_host_blocks() == 0
    """)


# A plan's memory serves another plan only once its own device has been waited for; the current device is what it was.
@pytest.mark.parametrize("failures,kept", [((0, 0, 0), True), ((1, 0, 0), False), ((0, 1, 0), False), ((0, 0, 1), False)])
@pytest.mark.parametrize("current", [0, 1])
def test_destroy_waits_for_the_plans_own_device(failures, kept, current):
    if current == 1 and failures == (1, 0, 0):
        kept = True                                        # nothing to select
    host_double.run("""
    D.hipSetDevice(1)
    plan = create(512, 3072, 768)
    assert D.double_blocks() == 1
    D.hipSetDevice(%d)
    D.double_forget()
    D.double_failures(*%r)
    assert L.fi_plan_destroy(plan) == 0
    D.double_failures(0, 0, 0)
    assert D.double_blocks() == %d and D.double_freed() == %d
    assert D.double_waited(1) == 1 or not %r
    now = C.c_int(-1)
    D.hipGetDevice(C.byref(now))
    assert now.value == %d
    """ % (current, failures, kept, not kept, kept, current))


# Room for what the largest batch with eight slots per tile row or more counts, 16384 trials, and not for more.
@pytest.mark.parametrize("M,N", [(512, 3072), (1000, 130), (64, 8192), (4096, 4096), (100000, 16)])
def test_parts_are_bounded_and_enough(M, N):
    host_double.run("""
    plan = create(%d, %d, 16)
    inject(plan, 1, OTHER)
    used = []
    for n in (1, 512, 513, 4000, 8192, 16384, 16385, 1000000):
        before = D.double_in_use()
        assert reserve(plan, n, SIDE) == 0
        used.append((n, D.double_in_use() - before - 24 * n))   # beside the six words of each trial
        for m in sorted({min(n, 100000), max(1, n // 300), min(n, 5000), min(n, 16384)}):
            D.double_forget()
            assert affected(plan, m, SIDE) == 0
            slots = D.double_launch_word([i for i, s in enumerate(names()) if "affected_element" in s][0], 0)
            assert parts_used() == (slots >= 8), (n, m, slots)
            assert slots < 8 or m <= 16384
        L.fi_plan_destroy(plan)
        fi.fi_release_memory()
        plan = create(%d, %d, 16)
        inject(plan, 1, OTHER)
    assert max(b for n, b in used) <= 4400000, used
    """ % (M, N, M, N))


# Items of four trials: up to six rounds of 512 resident workgroups of eight trials' items, with outputs and for the operand
# faults, whose launch is the second one then, up to 100 rounds x k-tiles.
@pytest.mark.parametrize("M,N,K,few,more,most", [(64, 2327, 160, 664, 2509, 3200), (128, 640, 144, 1224, 1232, 6824), (640, 640, 4096, 56, 64, 72)])
@pytest.mark.parametrize("outputs", [False, True])
def test_which_batches_run_four_trials_an_item(M, N, K, few, more, most, outputs):
    host_double.run("""
    M, N, K, outputs = %d, %d, %d, %r
    plan = create(M, N, K)
    tiles, k_tiles = -(-M // 64) * -(-N // 64), -(-K // 64)
    for n in (%d, %d, %d):
        items = tiles * -(-n // 8)
        D.double_forget()
        assert L.fi_gemm_inject_batch(plan, C.c_void_p(ANY), n, 1, C.c_void_p(ANY), C.c_void_p(ANY) if outputs else None, None) == 0
        run = [s for s in names() if "gemm_fi_" in s]
        kinds = ["four" if "gemm_fi_four" in s else "eight" if "gemm_fi_multi" in s else s for s in run]
        within = items * k_tiles <= 100 * 512
        want = ["eight", "eight"] if not within else ["four"] if outputs or items <= 6 * 512 else ["eight", "four"]
        assert kinds == want, (n, run)
        buf = C.create_string_buffer(1024)
        L.fi_plan_describe(plan, buf, 1024)
        lines = 8 * min(6 * 512 // tiles, 100 * 512 // (tiles * k_tiles)), 8 * (100 * 512 // (tiles * k_tiles))
        assert "at most %%d trials, operand faults and batches with outputs %%d: gemm_fi_four" %% lines in buf.value.decode(), buf.value
    """ % (M, N, K, outputs, few, more, most))
