"""The work by which the speed of this library is judged: named cases, a generator of more of them, and for each
case its inputs, one pass through the public entry points, the work it cannot do without and the accuracy it owes.

Three kinds of case.
  stage      one training step of a pipeline rank: gradients cleared, then po_run_schedule over all microbatches
             (forward, offload, reload, backward), as harness.StageRunner drives it.  The five named workloads C1-C5
             of inputs.CONFIGS give the widths; layer and microbatch counts are cut where the full workload would
             only repeat the same passes.
  attention  causal attention forward and backward on their own (po_op_attention_*).
  rows       the row-wise operations on their own: LayerNorm forward and backward, a bias gradient, dropout.
"""
from __future__ import annotations

import math
import weakref

import torch

from paper_2503_01328_amd import binding as po
from paper_2503_01328_amd import inputs as syn
from paper_2503_01328_amd.harness import StageRunner

SCHEDULES = {"1f1b": po.PO_SCHED_1F1B, "interleaved": po.PO_SCHED_1F1B_INTERLEAVED, "gis": po.PO_SCHED_GIS,
             "po": po.PO_SCHED_PO}

_STAGE_DEFAULTS = dict(kind="stage", chunks=1, kv_heads=0, vocab=0, dtype="bf16", schedule="1f1b", ratio=0.0, degree=4,
                       dropout=0.0, longest_lifespan=False, prefetch=2)


def _stage(name=None, **kw):
    case = dict(_STAGE_DEFAULTS, **kw)
    return case if name is None else dict(name=name, **case)


def listed():
    return [
        # Workload C1 as it is: the debugging configuration in fp32 with token and position embedding, every unit
        # offloaded.  Two hundred tiny launches: latency and host work.
        _stage("c1_fp32_embedding", layers=2, hidden=256, heads=4, ffn=1024, seq=128, micro=4, degree=2, vocab=1024,
               dtype="f32", ratio=1.0),
        # A reduced bf16 stage, the size a user brings a model up with (head size 64).
        _stage("small_bf16", layers=2, hidden=512, heads=8, ffn=2048, seq=512, micro=4, degree=2),
        # C2's widths on short prompts: few rows against full-width weights.
        _stage("short_rows_bf16", layers=2, hidden=2048, heads=16, ffn=8192, seq=100, micro=2),
        # C2's widths on a sequence that is no multiple of anything: unpadded documents.
        _stage("ragged_bf16", layers=2, hidden=2048, heads=16, ffn=8192, seq=1733, micro=2),
        # An ordinary fp32 stage: numerical debugging of a model of moderate width.
        _stage("wide_fp32", layers=2, hidden=1024, heads=16, ffn=4096, seq=1024, micro=2, dtype="f32"),
        # Workload C2 without offload: compute alone.
        _stage("c2_resident", layers=4, hidden=2048, heads=16, ffn=8192, seq=2048, micro=8),
        # Workload C2 with every unit offloaded: the benchmark's headline, bound by the host link.
        _stage("c2_full_offload", layers=4, hidden=2048, heads=16, ffn=8192, seq=2048, micro=8, ratio=1.0),
        # C3's widths with grouped-query attention, every other microbatch offloaded.
        _stage("c3_grouped_half_offload", layers=2, hidden=4096, heads=32, kv_heads=8, ffn=16384, seq=4096, micro=4,
               ratio=0.5),
        # C4's widths, two chunks, uniformly repeated schedule with split backward, dropout, the longest-lived chunk
        # of every microbatch offloaded.
        _stage("c4_split_backward", layers=2, chunks=2, hidden=4096, heads=32, ffn=16384, seq=4096, micro=8,
               schedule="po", ratio=0.5, longest_lifespan=True, prefetch=4, dropout=0.1),
        # C5's widths: long context, attention a third of the work.
        _stage("c5_long_context", layers=1, hidden=5120, heads=40, ffn=20480, seq=16384, micro=2, degree=2),
        # Attention alone, grouped heads of size 64, a sequence that ends inside a tile.
        dict(name="attention_ragged_grouped", kind="attention", seq=3000, heads=32, kv_heads=8, head_size=64,
             dtype="bf16"),
        # The row-wise operations at C5's width and an odd number of rows.
        dict(name="rows_bf16", kind="rows", rows=5001, hidden=5120, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Flops weighted by how far below the matrix-core rate the case's type and shape run."""
    gemm, attn = _stage_flops(c)
    matrix = c["dtype"] == "bf16" and c["seq"] % 128 == 0
    return (1 if matrix and all(w % 128 == 0 for w in (c["hidden"], c["ffn"], _qkv_width(c))) else 60) * gemm + \
        (1 if matrix else 600) * attn


def draw(rng):
    kind = rng.choices(["stage", "attention", "rows"], [8, 1, 1])[0]
    dtype = rng.choices(["bf16", "f32"], [4, 1])[0]
    if kind == "rows":
        return dict(kind="rows", rows=_log_int(rng, 100, 20000), hidden=64 * _log_int(rng, 4, 80), dtype=dtype)
    head_size = rng.choice([64, 128])
    if kind == "attention":
        heads = _log_int(rng, 2, 40)
        seq = _log_int(rng, 100, min(4000, int(math.sqrt(2e10 / (heads * head_size)))))
        if rng.random() < 0.5:
            seq = 128 * max(1, seq // 128)
        group = rng.choice([g for g in (1, 1, 2, 4, 8) if heads % g == 0])
        return dict(kind="attention", seq=seq, heads=heads, kv_heads=heads // group, head_size=head_size, dtype=dtype)
    heads = _log_int(rng, 2, 5120 // head_size)
    hidden = heads * head_size
    seq = _log_int(rng, 64, 16384)
    if rng.random() < 0.5:
        seq = 128 * max(1, seq // 128)
    schedule = rng.choice(["1f1b", "1f1b", "interleaved", "gis", "po"])
    chunks = 1 if schedule == "1f1b" else 2
    degree = rng.choice([2, 4])
    group = rng.choice([g for g in (1, 1, 2, 4, 8) if heads % g == 0])
    case = _stage(layers=chunks * rng.choice([1, 2]), chunks=chunks, hidden=hidden, heads=heads,
                  kv_heads=heads // group if group > 1 else 0, ffn=hidden * rng.choice([4, 4, 3, 2]), seq=seq,
                  micro=degree * rng.choice([1, 2]), degree=degree, dtype=dtype, schedule=schedule,
                  ratio=rng.choice([0.0, 0.0, 0.5, 1.0]), vocab=rng.choice([0, 0, 0, 2000]),
                  dropout=rng.choice([0.0, 0.0, 0.1]), longest_lifespan=rng.random() < 0.5)
    limit = 7e13
    while _cost(case) > limit:  # fewer repeats of the same passes first, then a shorter sequence
        if case["layers"] > chunks:
            case["layers"] = chunks
        elif case["micro"] > degree:
            case["micro"] = degree
        elif degree == 4:
            degree = case["degree"] = case["micro"] = 2
        else:
            seq = int(case["seq"] * 0.7)
            case["seq"] = 128 * max(1, seq // 128) if case["seq"] % 128 == 0 else seq
    return case


# ---- inputs -------------------------------------------------------------------------------------------------------
class _StageState:
    """A stage with its parameters, gradients, unit inputs and outputs; the stage goes when the state does."""

    def __init__(self, case, seed):
        shape = syn.StageShape(case["layers"], case["chunks"], case["hidden"], case["heads"], case["ffn"], case["seq"],
                               vocab=case["vocab"], dtype=case["dtype"], pipeline_degree=case["degree"],
                               n_microbatches=case["micro"], n_kv_heads=case["kv_heads"])
        self.runner = StageRunner(shape, seed=seed, device_params=True, dropout_p=case["dropout"], dropout_seed=1234,
                                  select_policy=int(case["longest_lifespan"]), prefetch_passes=case["prefetch"])
        self.runner.make_inputs_on_device(seed)
        self.schedule, self.ratio = SCHEDULES[case["schedule"]], case["ratio"]
        weakref.finalize(self, self.runner.close)


def _generator(seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return g


def _dtype(case):
    return (po.PO_BF16, torch.bfloat16) if case["dtype"] == "bf16" else (po.PO_F32, torch.float32)


def prepare(case, seed):
    if case["kind"] == "stage":
        return _StageState(case, seed)
    g = _generator(seed)
    code, dt = _dtype(case)
    rand = lambda *size: torch.randn(*size, generator=g, device="cuda:0").to(dt)
    if case["kind"] == "attention":
        s, h, hkv = case["seq"], case["heads"] * case["head_size"], case["kv_heads"] * case["head_size"]
        empty = lambda *size, t=dt: torch.empty(*size, dtype=t, device="cuda:0")
        return dict(case=case, code=code, qkv=rand(s, h + 2 * hkv), d_o=rand(s, h), o=empty(s, h),
                    lse=empty(case["heads"], s, t=torch.float32), dqkv=empty(s, h + 2 * hkv),
                    delta=empty(case["heads"], s, t=torch.float32),
                    partials=empty(s, 2 * h) if hkv < h else None)
    rows, h = case["rows"], case["hidden"]
    words = max(po.po_op_layernorm_backward_workspace(rows, h), po.po_op_colsum_workspace(rows, h)) // 4
    return dict(case=case, code=code, x=rand(rows, h), gain=1 + 0.02 * rand(h), shift=0.02 * rand(h), dn=rand(rows, h),
                dres=rand(rows, h), y=torch.empty(rows, h, dtype=dt, device="cuda:0"),
                dx=torch.empty(rows, h, dtype=dt, device="cuda:0"),
                dropped=torch.empty(rows, h, dtype=dt, device="cuda:0"),
                grads=torch.zeros(3, h, device="cuda:0"), workspace=torch.empty(words, device="cuda:0"))


# ---- one pass -----------------------------------------------------------------------------------------------------
def run(state):
    if isinstance(state, _StageState):
        r = state.runner
        r.grads.zero_()
        r.run(state.schedule, state.ratio)
        return {"y": r.y, "dx": [t for t in r.dx if t is not None], "grads": r.grads}
    case, code = state["case"], state["code"]
    if case["kind"] == "attention":
        s, h, a, akv = case["seq"], case["heads"] * case["head_size"], case["heads"], case["kv_heads"]
        po.po_op_attention_forward(code, state["qkv"], state["o"], state["lse"], s, h, a, n_kv_heads=akv)
        po.po_op_attention_backward(code, state["qkv"], state["o"], state["lse"], state["d_o"], state["dqkv"],
                                    state["delta"], s, h, a, n_kv_heads=akv, partials=state["partials"])
        return {"o": state["o"], "lse": state["lse"], "dqkv": state["dqkv"]}
    rows, h = case["rows"], case["hidden"]
    state["grads"].zero_()
    po.po_op_layernorm_forward(code, state["x"], state["gain"], state["shift"], state["y"], rows, h, 1e-5)
    po.po_op_dropout(code, state["dn"], state["dropped"], rows, h, 0.1, 1234, 0, 0, 0)
    po.po_op_colsum_accumulate(code, state["dropped"], state["grads"][2], state["workspace"], rows, h)
    po.po_op_layernorm_backward(code, state["dropped"], state["x"], state["gain"], state["dres"], state["dx"],
                                state["grads"][0], state["grads"][1], state["workspace"], rows, h, 1e-5)
    return {"y": state["y"], "dropped": state["dropped"], "dx": state["dx"], "grads": state["grads"]}


# ---- work ---------------------------------------------------------------------------------------------------------
def _qkv_width(case):
    return case["hidden"] + 2 * (case["kv_heads"] or case["heads"]) * (case["hidden"] // case["heads"])


def _stage_flops(case):
    """(matrix products, attention) of one step: forward, input gradient and weight gradient of the four projections;
    causal attention forward and backward."""
    s, h, f = case["seq"], case["hidden"], case["ffn"]
    passes = case["layers"] // case["chunks"] * case["chunks"] * case["micro"]
    return passes * 3 * 2 * s * h * (_qkv_width(case) + h + 2 * f), passes * 6 * s * s * h


def work(case):
    size = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "attention":
        s, h, hkv = case["seq"], case["heads"] * case["head_size"], case["kv_heads"] * case["head_size"]
        # q, k, v and d_o in, their gradients and o out
        return {"bytes": size * s * (2 * (h + 2 * hkv) + 2 * h) + 4 * case["heads"] * s, "flops": 6 * s * s * h}
    if case["kind"] == "rows":
        n = case["rows"] * case["hidden"]
        return {"bytes": size * 6 * n, "flops": 30 * n}  # x, dn, dres in; y, dropped, dx out
    s, h, f, L = case["seq"], case["hidden"], case["ffn"], case["layers"]
    params = L * (h * (_qkv_width(case) + h + 2 * f) + 6 * h + f + _qkv_width(case)) + (case["vocab"] + s) * h * bool(case["vocab"])
    units = case["micro"] * case["chunks"]
    moved = int(case["ratio"] * units)  # units that leave for the host and come back: their saved set is read and written
    saved = L // case["chunks"] * (s * (3 * h + _qkv_width(case) + f) * size + 4 * case["heads"] * s)
    gemm, attn = _stage_flops(case)
    return {"bytes": params * (size + 4) + units * 4 * s * h * size + 2 * moved * saved, "flops": gemm + attn}


def tolerance(case):
    """About four times the relative error (2-norm) measured against a computation at higher precision: bf16 stages
    of two to four layers 3.4e-3 to 6.5e-3 (against the same stage in fp32), fp32 stages 7e-7 (fp64 oracle); attention
    2.8e-3 and 7e-7, row-wise operations 1.7e-3 and 2e-7 (fp64)."""
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "rows":
        return {"rel": 7e-3 if bf16 else 1e-6}
    if case["kind"] == "attention":
        return {"rel": 1e-2 if bf16 else 3e-6}
    return {"rel": 2e-2 if bf16 else 6e-6}
