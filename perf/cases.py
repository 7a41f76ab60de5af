"""Performance cases of the fault-injection campaigns: what a user of this package has it do,
through its public entry points, over the range of sizes, formats, fault kinds and policies.

A case is one of five programs:

  campaign  a batch of trials on a plan that the program keeps: every trial recomputes the whole
            GEMM with its own fault; then the outcome classes (and, for product-term faults, the
            deviation histogram).
  affected  the same batch restricted to what each fault can reach (trials per second).
  layer     one layer of a sweep over a model's layers: a plan for its operands, a few trials with
            their corrected outputs, the classes, the plan given back.
  chain     the two-layer block Y = relu(X W1) W2: faults in layer 1 with the activations handed
            on in the operand format, then layer 2 on every trial's own activations.
  outputs   raw faulty outputs materialised, the stand-alone detector / corrector run over them,
            and the corrected outputs turned into the next layer's operand.

The five campaigns' shapes and value distributions are those of the package's own workloads;
here the inputs are drawn on the GPU.
"""
import torch

from paper_2311_05782_amd import fi

BASE = {"b_layout": 0, "bound": fi.BOUND_ROWCOL, "check": fi.PCHECK_NONE, "nbits": 1, "H": 0}


def _case(name, do, M, N, K, kb, fmt, trials, kind, policy, values, **more):
    return dict(BASE, name=name, do=do, M=M, N=N, K=K, kb=kb, fmt=fmt, trials=trials, kind=kind, policy=policy,
                values=values, **more)


def listed():
    return [
        # The smallest campaign, a unit test's or a tutorial's: launches and latency.
        _case("tiny_campaign", "campaign", 128, 128, 128, 32, fi.FP16, 64, fi.KIND_ALL_ACC, fi.CORRECT_ZERO, "normal"),
        # The paper's own fault with an exponent check on an odd-sized layer, weights stored K-major,
        # K not a multiple of the 64-wide k-tile, a handful of trials: a look at one layer.
        _case("product_few_ragged", "campaign", 300, 203, 176, 16, fi.BF16, 24, fi.KIND_ALL_PRODUCT, fi.CORRECT_ZERO,
              "relu", b_layout=1, check=fi.PCHECK_RANGE_MAX, nbits=4),
        # A transformer's linear layer, accumulator and activation faults mixed.
        _case("bert_campaign", "campaign", 512, 3072, 768, 32, fi.FP16, 4096, fi.KIND_MIX_ACC_A, fi.CORRECT_RECOMPUTE,
              "weights"),
        # A convolution as a GEMM: tall, narrow, half of the activations zero.
        _case("conv_campaign", "campaign", 3136, 64, 576, 32, fi.BF16, 8192, fi.KIND_ALL_ACC, fi.CORRECT_ZERO, "relu"),
        # Weight faults in a layer none of whose sizes fits a tile.
        _case("ragged_campaign", "campaign", 1000, 1010, 1008, 16, fi.FP16, 512, fi.KIND_ALL_B, fi.CORRECT_RECOMPUTE,
              "weights"),
        # Many two-bit trials on rows of very different magnitude: the detector's coverage.
        _case("stress_campaign", "campaign", 1024, 1024, 1024, 32, fi.FP16, 16384, fi.KIND_ALL_ACC, fi.CORRECT_ZERO,
              "heavy", nbits=2),
        # The largest: the headline batch.
        _case("square_campaign", "campaign", 4096, 4096, 4096, 64, fi.BF16, 1024, fi.KIND_ALL_ACC, fi.CORRECT_ZERO,
              "uniform"),
        # Outcome statistics at many trials per second: only what a fault reaches is computed.
        _case("bert_affected", "affected", 512, 3072, 768, 32, fi.FP16, 4096, fi.KIND_MIX_ACC_A, fi.CORRECT_RECOMPUTE,
              "weights"),
        _case("square_affected", "affected", 4096, 4096, 4096, 64, fi.BF16, 1024, fi.KIND_ALL_ACC, fi.CORRECT_ZERO,
              "uniform"),
        # One step of a sweep over layers.
        _case("bert_layer", "layer", 512, 3072, 768, 32, fi.BF16, 8, fi.KIND_ALL_ACC, fi.CORRECT_ZERO, "weights"),
        # A feed-forward block, 512 tokens, 768 -> 3072 -> 768.
        _case("mlp_chain", "chain", 512, 768, 768, 32, fi.BF16, 256, fi.KIND_ALL_ACC, fi.CORRECT_ZERO, "weights",
              H=3072),
        # Materialised outputs of the convolution.
        _case("conv_outputs", "outputs", 3136, 64, 576, 32, fi.BF16, 128, fi.KIND_ALL_ACC, fi.CORRECT_ZERO, "relu"),
    ]


MOST_FLOPS = 3e13      # of a drawn case: a fifth of the largest listed one's
MOST_OUTPUTS = 3e7     # materialised elements of a drawn case


def draw(rng):
    def spread(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    do = rng.choice(["campaign", "campaign", "affected", "layer", "chain", "outputs"])
    fmt = rng.choice([fi.FP16, fi.BF16])
    M, N, K = spread(16, 4096), spread(16, 4096), 16 * spread(2, 256)
    H = 0
    if do == "chain":
        K, H, N = 64 * spread(1, 32), 64 * spread(1, 64), 8 * spread(2, 256)
    kb = rng.choice([b for b in (16, 32, 64) if K % b == 0 and H % b == 0])
    kind = rng.choice([fi.KIND_ALL_ACC, fi.KIND_ALL_A, fi.KIND_ALL_B, fi.KIND_MIX_ACC_A, fi.KIND_ALL_PRODUCT])
    each = 2.0 * M * N * K if do != "chain" else 2.0 * M * H * (K + N)
    most = MOST_FLOPS / each
    if do == "affected":
        most = 16384
    if do in ("layer", "outputs"):
        most = min(most, MOST_OUTPUTS / (M * N))
    if do == "chain":
        most = min(most, MOST_OUTPUTS / (M * H))
    top = max(2, min(16384 if do in ("campaign", "affected") else 64 if do == "layer" else 256, int(most)))
    return dict(BASE, do=do, M=M, N=N, K=K, kb=kb, fmt=fmt, H=H, trials=spread(2, top), kind=kind,
                policy=rng.choice([fi.CORRECT_ZERO, fi.CORRECT_RECOMPUTE]),
                values=rng.choice(["normal", "weights", "relu", "uniform", "heavy"]),
                b_layout=rng.choice([0, 0, 1]), bound=rng.choice([fi.BOUND_ROWCOL, fi.BOUND_ROWCOL, fi.BOUND_GLOBAL]),
                nbits=rng.choice([1, 2, 4]),
                check=rng.choice([fi.PCHECK_NONE, fi.PCHECK_BOUND, fi.PCHECK_RANGE_MAX, fi.PCHECK_RANGE_FLIP])
                if kind == fi.KIND_ALL_PRODUCT else fi.PCHECK_NONE)


def _type(case):
    return torch.float16 if case["fmt"] == fi.FP16 else torch.bfloat16


def _operands(case, seed):
    """A [M][K] and B as case["b_layout"] stores it ([N][K] or [K][N]), in the operand format; for a
    chain also the second weight matrix [N][H], with H in the place of N in the first."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    M, K, values = case["M"], case["K"], case["values"]
    N = case["H"] or case["N"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    if values == "uniform":
        a = torch.rand(M, K, generator=g, device="cuda") * 2 - 1
        b = torch.rand(N, K, generator=g, device="cuda") * 2 - 1
    else:
        a, b = normal(M, K), normal(N, K)
        if values == "relu":
            a, b = a.clamp_min(0), b * (2.0 / K) ** 0.5
        elif values == "weights":
            b = b * 0.02
        elif values == "heavy":
            a[torch.randperm(M, generator=g, device="cuda")[:max(1, round(0.2 * M))]] *= 100
    t = _type(case)
    ops = [a.to(t), (b if case["b_layout"] == 0 else b.t().contiguous()).to(t)]
    if case["H"]:
        ops.append((normal(case["N"], case["H"]) * 0.02).to(t))
    return ops


def _desc(case, M, N, K, b_layout=0):
    return fi.plan_desc(M, N, K, case["kb"], case["fmt"], b_layout=b_layout, bound_mode=case["bound"])


class _Records:
    """The records of a batch and what is computed from them, as tensors."""

    def __init__(self, n, faults=None):
        self.n = n
        self.raw = fi.empty_results(n)
        words = self.raw.view(torch.int32).view(n, 12)
        self.classes = torch.empty(n, dtype=torch.uint8, device="cuda")
        self.totals = torch.empty(3, dtype=torch.int64, device="cuda")
        self.out = {"counters": words[:, 0:4], "largest": words[:, 4:6].view(torch.float32), "words": words[:, 6:12],
                    "classes": self.classes, "totals": self.totals}

    def classify(self, plan):
        plan.fi_classify(self.raw, self.n, self.classes, self.totals)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, s.n, s.policy = case, case["trials"], case["policy"]
    M, N, K, H, n, do = case["M"], case["N"], case["K"], case["H"], case["trials"], case["do"]
    s.ops = _operands(case, seed)
    s.desc = _desc(case, M, H or N, K, case["b_layout"])
    faults = fi.fi_sample_faults(seed, 0, n, s.desc, case["kind"], case["nbits"])
    if do in ("layer", "chain", "outputs"):
        faults["kind"][0] = fi.SITE_NONE      # the fault-free run that the others are looked at against
    s.faults = fi.to_device(faults)
    s.rec = _Records(n)
    s.plan = None
    if do != "layer":
        s.plan = fi.Plan(s.desc, s.ops[0], s.ops[1])
        s.plan.set_product_check(case["check"])
        s.plan.reserve(n)
    s.out = dict(s.rec.out)
    s.hist = None
    if do in ("campaign", "affected") and case["kind"] == fi.KIND_ALL_PRODUCT:
        s.hist = s.out["histogram"] = torch.empty(256, dtype=torch.int64, device="cuda")
    if do in ("layer", "outputs"):
        s.c = torch.empty(n, M, N, device="cuda")
        s.out.update(fault_free=s.c[0], faulty=s.c[1:])
    if do == "outputs":
        s.flags = torch.empty(n, M, N, dtype=torch.uint8, device="cuda")
        s.flagged = torch.empty(n, dtype=torch.int32, device="cuda")
        s.h = torch.empty(n, M, N, dtype=_type(case), device="cuda")
        s.out.update(flags=s.flags, flagged=s.flagged, handed_on=s.h[0], handed_on_faulty=s.h[1:])
    if do == "chain":
        s.h = torch.empty(n, M, H, dtype=_type(case), device="cuda")
        # layer 2's plan is made for the fault-free activations
        s.plan.fi_gemm_inject_batch_act(s.faults, 1, s.policy, s.rec.raw, s.h)
        s.h_clean = s.h[0].clone()
        s.plan2 = fi.Plan(_desc(case, M, N, H), s.h_clean, s.ops[2])
        s.rec2 = _Records(n)
        s.out = {"layer1": s.rec.out["counters"], "handed_on": s.h[0], "handed_on_faulty": s.h[1:], "layer2": s.rec2.out}
    return s


def run(s):
    do = s.case["do"]
    if do == "campaign" or do == "affected":
        if do == "campaign":
            s.plan.fi_gemm_inject_batch(s.faults, s.n, s.policy, s.rec.raw)
        else:
            s.plan.fi_gemm_inject_batch_affected(s.faults, s.n, s.policy, s.rec.raw)
        s.rec.classify(s.plan)
        if s.hist is not None:
            s.plan.fi_deviation_histogram(s.faults, s.rec.raw, s.n, fi.HIST_SITE, s.hist)
    elif do == "layer":
        plan = fi.Plan(s.desc, s.ops[0], s.ops[1])
        plan.set_product_check(s.case["check"])
        plan.fi_gemm_inject_batch(s.faults, s.n, s.policy, s.rec.raw, s.c)
        s.rec.classify(plan)
        plan.destroy()
    elif do == "chain":
        s.plan.fi_gemm_inject_batch_act(s.faults, s.n, s.policy, s.rec.raw, s.h)
        s.plan2.fi_gemm_propagate_batch(s.h, s.h[0].numel(), s.n, s.policy, s.rec2.raw)
        s.rec2.classify(s.plan2)
    else:
        s.plan.fi_gemm_inject_batch(s.faults, s.n, fi.CORRECT_NONE, s.rec.raw, s.c)
        s.plan.fi_detect_correct(s.c, s.n, s.policy, s.flags, s.flagged)
        fi.fi_activation_round(s.case["fmt"], s.c, s.c.numel(), s.h)
        s.rec.classify(s.plan)
    return s.out


def work(case):
    """Every trial of a campaign executes its whole GEMM; an affected trial its element, row or
    column.  Operands, faults and records are read or written once, and the outputs asked for."""
    M, N, K, H, n, do = case["M"], case["N"], case["K"], case["H"], case["trials"], case["do"]
    records = (20.0 + 48.0 + 1.0) * n
    if do == "chain":
        return {"flops": 2.0 * M * H * (K + N) * n,
                "bytes": 2.0 * (M * K + H * K + N * H + M * H) + 4.0 * M * H * n + records + 49.0 * n}
    operands = 2.0 * (M * K + N * K)
    if do == "affected":
        row, col = float(N), float(M)
        reach = {fi.KIND_ALL_A: row, fi.KIND_ALL_B: col, fi.KIND_MIX_ACC_A: (1 + row) / 2}.get(case["kind"], 1.0)
        touched = n * 2.0 * K * (1 + reach)       # operand bytes, if no two trials shared any
        return {"flops": 2.0 * K * reach * n, "bytes": min(operands, touched) + records + min(8.0 * M * N, 8.0 * reach * n)}
    flops = 2.0 * M * N * K * n
    if do == "layer":                             # the fault-free result and the magnitude sums too
        return {"flops": flops + 4.0 * M * N * K, "bytes": operands + records + 8.0 * M * N + 4.0 * M * N * n}
    if do == "outputs":
        return {"flops": flops, "bytes": operands + records + (4.0 + 1.0 + 2.0) * M * N * n}
    return {"flops": flops, "bytes": operands + records}


def tolerance(case):
    """Records, classes and outputs are the same bits from one run to the next and for every tile
    shape: each output element is accumulated by the same sequence of 16-wide matrix steps."""
    return "exact"


def exact(case, seed):
    """The fault-free trial in 64 bits, where its outputs are asked for; a faulty accumulator's
    bits have no value in other arithmetic, and counters and classes are whole numbers."""
    do = case["do"]
    if do not in ("layer", "chain", "outputs"):
        return None
    ops = [x.double() for x in _operands(case, seed)]
    c = ops[0] @ (ops[1].t() if case["b_layout"] == 0 else ops[1])
    if do == "chain":
        return {"handed_on": c.clamp_min(0)}
    out = {"fault_free": c}
    if do == "outputs":
        out["handed_on"] = c.clamp_min(0)
    return out
