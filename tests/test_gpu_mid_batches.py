"""Batches between the smallest and the largest: four trials per item, the operand faults behind the other trials in
one launch.  Against the shapes that fi_plan_tune chooses (one trial per workgroup; eight trials, two launches), byte for
byte."""
import numpy as np
import pytest

from oracle import pyoracle as orc
from paper_2311_05782_amd import fi, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def _faults(plan, n, operand):
    """n faults of which every `operand`-th (0: none, 1: all) is an operand fault, with fault-free and invalid ones."""
    f = fi.fi_sample_faults(3, 0, n, plan.desc, fi.KIND_ALL_ACC, 2)
    f[1::3] = fi.fi_sample_faults(4, 0, n, plan.desc, fi.KIND_ALL_PRODUCT, 4)[1::3]
    f[::7]["kind"] = fi.SITE_NONE
    f[5::11]["row"] = 10 ** 7
    if operand:
        for k, kind in enumerate((fi.KIND_ALL_A, fi.KIND_ALL_B)):
            f[k * operand::2 * operand] = fi.fi_sample_faults(5 + k, 0, n, plan.desc, kind, 1)[k * operand::2 * operand]
    return f


# (M, N, K, k-block), trials, every how many-th is an operand fault.  The first part ends 1 .. 8 trials into a group of
# eight, so that the descriptors' padding holds a group of four or none, and either part may be empty; ragged tiles
# and k-tiles, an odd number of k-tiles, the shortest K; the longest batch that one step of the partition kernel sees; two
# items per workgroup, several from the counters, more than six rounds of eights, of which only the operand faults (some, none,
# all) run in fours, and 64 or more (99000 trials), where workgroups look into other XCDs' slices.
@pytest.mark.parametrize("shape,n,operand", [
    ((300, 300, 512, 32), 121, 0), ((300, 300, 512, 32), 124, 1), ((300, 300, 512, 32), 127, 5), ((320, 256, 512, 32), 260, 2),
    ((300, 300, 512, 32), 133, 132), ((129, 515, 464, 16), 205, 3), ((1000, 130, 320, 32), 119, 4),
    ((250, 1000, 80, 16), 440, 3), ((600, 300, 192, 32), 900, 6), ((600, 300, 192, 32), 901, 0), ((600, 300, 192, 32), 905, 1), ((300, 300, 512, 32), 1024, 3), ((300, 300, 512, 32), 1025, 4), ((70, 60, 128, 32), 50001, 9), ((70, 60, 128, 32), 99000, 9),
])
def test_mid_batches_equal_the_other_shapes(shape, n, operand):
    import torch
    M, N, K, kb = shape
    fmt = orc.FP16 if n % 2 else orc.BF16
    Aw, Bw = wl.gaussian(M, N, K, fmt, seed=n)
    plan, eight = gu.make_plan(Aw, Bw, kb, fmt), gu.make_plan(Aw, Bw, kb, fmt, cfg=6)
    # the library's own lines: eight trials of a 64 x 64 tile, two workgroups per compute unit; more steps and tiles per
    # SIMD than the small kernel takes
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = -(-M // 32) * -(-N // 32)
    assert n * tiles * (K // 16) / (4 * cus) + 15 * ((n + 3) // 4 * 4) * tiles / (4 * cus) > 550
    assert -(-M // 64) * -(-N // 64) * -(-n // 8) * -(-K // 64) <= 100 * 2 * cus and K > 64
    if n == 99000:
        assert -(-M // 64) * -(-N // 64) * (n // 4) / (3 * (cus // 8 * 8)) >= 64
    faults = _faults(plan, n, operand)
    want = gu.gpu_campaign(eight, faults, wl.CORRECT_RECOMPUTE)
    d_f = fi.to_device(faults)
    for _ in range(2):
        d_r = fi.empty_results(n).fill_(0xFF)           # the records are cleared by the call
        plan.fi_gemm_inject_batch(d_f, n, wl.CORRECT_RECOMPUTE, d_r)
        got = fi.results_to_host(d_r)
        assert got.tobytes() == want.tobytes(), [t for t in range(n) if got[t] != want[t]][:5]
    def with_half_outputs():
        outs = []
        for p in (plan, eight):
            d_r, d_h = fi.empty_results(n), torch.zeros((n, M, N), dtype=torch.int16, device="cuda")
            p.fi_gemm_inject_batch_act(d_f, n, wl.CORRECT_ZERO, d_r, d_h)
            outs.append((fi.results_to_host(d_r).tobytes(), d_h))
        assert outs[0][0] == outs[1][0] and torch.equal(outs[0][1], outs[1][1])
    with_half_outputs()                                   # without outputs the larger batches run in two launches
    if n < 1000:
        one = gu.make_plan(Aw, Bw, kb, fmt, cfg=2)
        r1, c1 = gu.gpu_campaign(one, faults, wl.CORRECT_ZERO, want_c=True)
        r4, c4 = gu.gpu_campaign(plan, faults, wl.CORRECT_ZERO, want_c=True)
        assert r1.tobytes() == r4.tobytes() and c1.tobytes() == c4.tobytes()
        one.destroy()
        # the entry point without allocations runs the same kernels
        d_r = fi.empty_results(n)
        plan.fi_gemm_inject_batch_noalloc(d_f, n, wl.CORRECT_RECOMPUTE, d_r)
        assert fi.results_to_host(d_r).tobytes() == want.tobytes()
    plan.destroy()
    eight.destroy()
