"""Performance cases: the fused subgraphs that a program hands to this library, from the smallest call to the largest.

A case names a pattern of `workloads` (its DAG is built there), its sizes and, where the pattern has a choice, the dtype of
the big tensors.  `prepare` makes the plan, loads it and makes the seeded device inputs; `run` enqueues the plan once on the
current stream.  `exact` evaluates the same DAG op by op in torch float64.
"""
import math

import torch

import paper_1811_05213_amd as fs
from paper_1811_05213_amd.runner import DeviceRun
from workloads import configs, patterns
from workloads.graph import FREE_OPS, min_hbm_bytes

DEVICE = "cuda:0"
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "u8": torch.uint8}

# pattern -> (graph builder, takes a dtype, largest drawn rows * cols, smallest and largest drawn cols)
PATTERNS = {
    "softmax": (configs.softmax_graph, False, 1 << 26, 16, 131072),
    "masked_softmax": (patterns.masked_softmax, True, 1 << 25, 16, 8192),
    "add_layernorm": (patterns.add_layernorm, True, 1 << 25, 64, 16384),
    "layernorm_gelu": (configs.layernorm_gelu_graph, False, 1 << 26, 64, 16384),
    "layernorm_grad": (configs.layernorm_grad_graph, False, 1 << 25, 64, 8192),
    "elementwise20": (configs.elementwise20_graph, False, 1 << 25, 16, 16384),
    "multi_reduce": (configs.multi_reduce_graph, False, 1 << 26, 16, 8192),
    "batchnorm": (patterns.batchnorm, False, 1 << 25, 16, 8192),
    "transpose": (patterns.transpose, True, 1 << 26, 16, 65536),
    "dropout_residual": (patterns.dropout_residual, True, 1 << 26, 16, 16384),
}


def listed():
    return [
        # the smallest call: a few attention heads' scores; latency of one launch
        {"name": "softmax f32 256x1024", "pattern": "softmax", "rows": 256, "cols": 1024},
        # one decoding step of a batch of 32: residual add and LayerNorm over one row per sequence
        {"name": "add_layernorm bf16 32x4096", "pattern": "add_layernorm", "rows": 32, "cols": 4096, "dtype": "bf16"},
        # a graph of fine-grained ops that splits into several launches: 200 nodes over [512, 64..256]
        {"name": "random_dag f32 512", "pattern": "random_dag", "rows": 512, "cols": 256},
        # the ordinary forward block of a training step or a prefill
        {"name": "layernorm_gelu bf16 16384x1024", "pattern": "layernorm_gelu", "rows": 16384, "cols": 1024},
        # prefill attention over 577 keys (a 24 x 24 grid and one more): an odd row length, padded rows
        {"name": "masked_softmax bf16 16384x577", "pattern": "masked_softmax", "rows": 16384, "cols": 577, "dtype": "bf16"},
        # the backward pass of LayerNorm: row and column reductions in one subgraph
        {"name": "layernorm_grad f32 8192x4096", "pattern": "layernorm_grad", "rows": 8192, "cols": 4096},
        # column statistics and row norms from one read
        {"name": "multi_reduce f32 65536x512", "pattern": "multi_reduce", "rows": 65536, "cols": 512},
        # training-mode batch normalisation: column statistics that every row needs again
        {"name": "batchnorm f32 16384x1024", "pattern": "batchnorm", "rows": 16384, "cols": 1024},
        # a layout change between two library calls
        {"name": "transpose bf16 16384x4096", "pattern": "transpose", "rows": 16384, "cols": 4096, "dtype": "bf16"},
        # dropout with a byte mask and the residual add
        {"name": "dropout_residual bf16 16384x4096", "pattern": "dropout_residual", "rows": 16384, "cols": 4096, "dtype": "bf16"},
        # the loss head: probabilities over a vocabulary of odd size
        {"name": "softmax f32 2048x50001", "pattern": "softmax", "rows": 2048, "cols": 50001},
        # the largest: a long elementwise chain over four 256 MiB inputs
        {"name": "elementwise20 f32 65536x1024", "pattern": "elementwise20", "rows": 65536, "cols": 1024},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pattern = rng.choice(sorted(PATTERNS) + ["random_dag"])
    if pattern == "random_dag":
        return {"pattern": pattern, "rows": _log_uniform(rng, 48, 2048), "cols": rng.choice([32, 48, 64, 100, 128, 200, 256, 384])}
    _, typed, most, lo, hi = PATTERNS[pattern]
    cols = _log_uniform(rng, lo, hi)
    if rng.random() < 0.5:  # as often as not the width is a round one
        cols = max(lo, (cols + 32) // 64 * 64)
    rows = max(1, min(65536, _log_uniform(rng, 1 << 13, most) // cols))
    case = {"pattern": pattern, "rows": rows, "cols": cols}
    if typed:
        case["dtype"] = rng.choice(["bf16", "f32"])
    return case


def _graph(case):
    if case["pattern"] == "random_dag":
        k = case["cols"]
        return configs.random_dag_graph(rows=case["rows"], ks=(k // 4, k // 2, k))
    build, typed = PATTERNS[case["pattern"]][:2]
    return build(case["rows"], case["cols"], case["dtype"]) if typed else build(case["rows"], case["cols"])


def _inputs(case, g, seed):
    """The plan's inputs on the GPU, from the seed alone: [rows, cols] tensors in the plan's dtypes."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    pattern, r, c = case["pattern"], case["rows"], case["cols"]
    out = []
    for k, i in enumerate(g.input_ids()):
        n = g.nodes[i]
        if n.dtype == "u8":  # nine of ten elements are kept
            t = (torch.rand((n.rows, n.cols), generator=gen, device=DEVICE) < 0.9).to(torch.uint8)
        elif pattern == "elementwise20":
            t = torch.rand((n.rows, n.cols), generator=gen, device=DEVICE)
            t = t * 4 - 2 if k < 4 else t * 2 - 1
        elif pattern == "masked_softmax" and k == 1:  # every row ends in padding: half of the keys at most
            keep = torch.randint((c + 1) // 2, c + 1, (r, 1), generator=gen, device=DEVICE)
            t = torch.where(torch.arange(c, device=DEVICE) < keep, 0.0, -30000.0)
        else:
            t = torch.randn((n.rows, n.cols), generator=gen, device=DEVICE)
            if pattern in ("multi_reduce", "batchnorm") and k == 0:
                t += 0.5
            elif pattern == "masked_softmax":
                t *= 8
            elif n.rows == 1 and pattern != "random_dag":
                first = k == min(j for j, i2 in enumerate(g.input_ids()) if g.nodes[i2].rows == 1)
                t = 1 + 0.1 * t if first else 0.1 * t  # a scale, then shifts
        out.append(t.to(_TORCH[n.dtype]))
    return out


def prepare(case, seed):
    g = _graph(case)
    r = DeviceRun(fs.Plan(g), DEVICE)
    r.plan.load()
    r.set_device_inputs(_inputs(case, g, seed))
    outputs = [t.view(torch.bfloat16) if n.dtype == "bf16" else t for t, n in zip(r.outputs, r.out_nodes)]
    return {"run": r, "outputs": outputs}


def run(state):
    state["run"].launch()
    return state["outputs"]


def work(case):
    g = _graph(case)
    flops = sum(g.nodes[i].rows * g.nodes[i].cols for i in g.compute_ids() if g.nodes[i].op not in ("transpose", "convert"))
    flops += sum(g.nodes[g.nodes[i].ins[0]].rows * g.nodes[g.nodes[i].ins[0]].cols for i in g.compute_ids() if g.nodes[i].op.startswith("reduce"))
    return {"bytes": min_hbm_bytes(g), "flops": flops}


def tolerance(case):
    """About four times what fused and one-op-per-launch execution of the same DAG differ by."""
    if case["pattern"] == "transpose":
        return "exact"
    if case["pattern"] == "random_dag":
        # chains of some tens of ops with row sums that cancel among them (7e-7 from float64 at the worst of ten sizes)
        return {"rel": 2e-6, "max": 2e-5}
    if case["pattern"] in ("masked_softmax", "add_layernorm", "layernorm_gelu", "dropout_residual") and case.get("dtype", "bf16") == "bf16":
        # a bf16 result rounds the other way (2^-7 of its value at most) where the fp32 value before it lies next to a midpoint
        return {"rel": 2e-4, "max": 1.6e-2}
    return {"rel": 8e-7, "max": 4e-6}


# ---------------------------------------------------------------------------------------------------------------------------
# the same DAG in float64
# ---------------------------------------------------------------------------------------------------------------------------
_UNARY = {"neg": torch.neg, "abs": torch.abs, "exp": torch.exp, "log": torch.log, "tanh": torch.tanh, "sigmoid": torch.sigmoid,
          "sqrt": torch.sqrt, "rsqrt": torch.rsqrt, "rcp": torch.reciprocal, "convert": lambda x: x,
          "gelu_tanh": lambda x: torch.nn.functional.gelu(x, approximate="tanh")}
_BINARY = {"add": torch.add, "sub": torch.sub, "mul": torch.mul, "div": torch.div, "max": torch.maximum, "min": torch.minimum}
_CMP = {"gt": torch.gt, "ge": torch.ge, "lt": torch.lt, "le": torch.le, "eq": torch.eq, "ne": torch.ne}
_REDUCE = {"sum": torch.sum, "mean": torch.mean, "max": torch.amax, "min": torch.amin}


def exact(case, seed):
    g = _graph(case)
    # what a comparison decides is part of the graph's definition: values it depends on are rounded to their dtype
    decides, stack = set(), [j for n in g.nodes if n.op == "cmp" for j in n.ins]
    while stack:
        i = stack.pop()
        if i not in decides:
            decides.add(i)
            stack += g.nodes[i].ins
    last = {}
    for i, n in enumerate(g.nodes):
        for j in n.ins:
            last[j] = i
    inputs = iter(_inputs(case, g, seed))
    val = {}
    for i, n in enumerate(g.nodes):
        a = [val[j] for j in n.ins]
        if n.op == "input":
            v = next(inputs)
            v = v if n.dtype == "u8" else v.double()
        elif n.op == "const":
            v = torch.tensor(n.value, dtype=torch.float32, device=DEVICE).double().expand(n.rows, n.cols)
        elif n.op in _UNARY:
            v = _UNARY[n.op](a[0])
        elif n.op in _BINARY:
            v = _BINARY[n.op](a[0], a[1])
        elif n.op == "cmp":
            v = _CMP[n.attr](a[0], a[1]).to(torch.uint8)
        elif n.op == "select":
            v = torch.where(a[0] != 0, a[1], a[2])
        elif n.op in ("bcast_rowvec", "bcast_colvec"):
            v = a[0].expand(n.rows, n.cols)
        elif n.op == "transpose":
            v = a[0].t()
        else:
            v = _REDUCE[n.attr](a[0], dim=1 if n.op == "reduce_row" else 0, keepdim=True)
        if i in decides and n.op not in FREE_OPS:
            v = v.to(_TORCH[n.dtype]).to(v.dtype)
        val[i] = v
        for j in n.ins:
            if last[j] == i and j not in g.outputs:
                val.pop(j, None)
    return [val[o].contiguous() for o in g.outputs]
