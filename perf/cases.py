"""The work that programs hand to this library, as cases whose time can be taken.

A case is a dict of plain values.  Four kinds of work, each through the public entry points:

  step       one CodedReduce iteration for a program with an optimiser of its own: cr_partial_grads, cr_encode_tree, cr_decode_root
  train      gradient descent kept on the device: one cr_gd_run call over several steps, from the initial model on
  aggregate  partial gradients made elsewhere: cr_load_partial_grads, cr_encode_tree, cr_decode_root; with several steps, every
             step with gradients of its own, one cr_aggregate_run call
  layers     the same for a network whose layers are handed over one after the other: one cr_aggregate_static call per layer

Trees and sizes are those of the benchmark workloads (cr_inputs/workloads.py), of the paper's experiments and of the tests.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1902_01981_amd as cr

# (L, n, s): the trees of the benchmark workloads and of the tests; depth, width, redundancy (1 to 27 holders per row) and codes vary
TREES = [(2, 3, 1), (2, 4, 1), (3, 4, 1), (3, 6, 2), (2, 8, 2), (2, 12, 1), (2, 12, 2), (3, 3, 1), (4, 2, 1), (1, 4, 2), (1, 6, 2),
         (1, 10, 4), (2, 4, 0), (1, 10, 0)]
# two convolutions and three dense layers, weights and biases: the network of the paper's simulated training, 117 706 parameters
LAYERS = [3 * 16 * 3 * 3, 16, 16 * 64 * 4 * 4, 64, 64 * 384, 384, 384 * 192, 192, 192 * 10, 10]


def _case(kind, tree, m, d, logistic=False, bf16=False, steps=1, measures=False):
    L, n, s = tree
    return {"kind": kind, "L": L, "n": n, "s": s, "m": m, "d": d, "logistic": logistic, "bf16": bf16, "steps": steps, "measures": measures}


def listed():
    return [
        # the smallest problem of the benchmark, an iteration at a time: launches and the calls themselves
        dict(_case("step", (2, 3, 1), 1_200, 100), name="step 1200x100"),
        # ... and a short training run on it with both convergence measures
        dict(_case("train", (2, 3, 1), 1_200, 100, steps=20, measures=True), name="train 1200x100"),
        # the paper's own linear regression on 84 workers: the data fit the last-level cache
        dict(_case("train", (3, 4, 1), 7_644, 6_500, steps=16), name="train 7644x6500"),
        # the size of the paper's logistic regression on its 156 workers, three stragglers in twelve: an odd number of columns
        dict(_case("step", (2, 12, 3), 6_552, 5_001, logistic=True), name="step 6552x5001 logistic"),
        # one layer of ten workers, bf16 rows that start on any 2-byte boundary
        dict(_case("step", (1, 10, 4), 60_000, 1_027, logistic=True, bf16=True), name="step 60000x1027 bf16"),
        # rows wider than one team of threads can hold in registers
        dict(_case("step", (2, 4, 1), 4_000, 50_008, logistic=True, bf16=True), name="step 4000x50008 bf16"),
        # the three large regressions of the benchmark: 4 GB of data each
        dict(_case("step", (2, 4, 1), 100_000, 10_000), name="step 100000x10000"),
        dict(_case("step", (3, 4, 1), 252_000, 4_096, logistic=True), name="step 252000x4096 logistic"),
        dict(_case("step", (3, 6, 2), 2_064_000, 1_024, bf16=True), name="step 2064000x1024 bf16"),
        # a network's gradients layer by layer, as a training framework hands them over: ten vectors of 10 to 73 728 entries
        dict(_case("layers", (2, 12, 2), 49_920, sum(LAYERS)), name="layers 117706"),
        # the same network's gradients as one vector, five stragglers in twelve, eight training steps
        dict(_case("aggregate", (2, 12, 5), 49_920, 117_706, steps=8), name="aggregate 8x117706"),
        # vectors of a large network: the largest aggregation of the benchmark
        dict(_case("aggregate", (2, 8, 2), 88, 1 << 24), name="aggregate 16777216"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    tree = rng.choice(TREES)
    workers = sum(tree[1] ** l for l in range(1, tree[0] + 1))
    kind = rng.choice(4 * ["step"] + 2 * ["train"] + 2 * ["aggregate"] + ["layers"])
    if kind == "layers":
        return _case("layers", rng.choice([(2, 12, 1), (2, 12, 2), (2, 4, 1), (1, 10, 4)]), rng.randint(2_000, 60_000), sum(LAYERS))
    if kind == "aggregate":
        steps = rng.choice([1, 1, 4, 8])
        m = rng.randint(workers, 40 * workers)
        slabs = 4 * workers                              # about as many vectors as such a tree has
        return _case("aggregate", tree, m, _log_uniform(rng, 64, min(1 << 24, 2_000_000_000 // (slabs * steps))), steps=steps)
    bf16 = rng.random() < 0.4
    steps = rng.choice([4, 8, 16]) if kind == "train" else 1
    d = _log_uniform(rng, 16, 60_000)
    m = min(4_000_000, max(2 * workers, _log_uniform(rng, 100_000, 1_000_000_000 // steps) // d))
    return _case(kind, tree, m, d, logistic=rng.random() < 0.4, bf16=bf16, steps=steps, measures=kind == "train" and rng.random() < 0.5)


def _masks(case, seed):
    """One straggler mask per step: in every sibling group a random set of s children, now and then fewer."""
    rng = np.random.default_rng([seed, 3])
    L, n, s = case["L"], case["n"], case["s"]
    groups = sum(n ** l for l in range(L))
    masks = np.zeros((case["steps"], groups * n), dtype=np.uint8)
    for t in range(case["steps"]):
        for g in range(groups):
            count = s if rng.random() < 0.9 else int(rng.integers(0, s + 1))
            masks[t, g * n + rng.choice(n, size=count, replace=False)] = 1
    return masks


def _plan(case, d=None, B=None):
    model = cr.CR_AGGREGATE_ONLY if case["kind"] in ("aggregate", "layers") else cr.CR_LOGISTIC if case["logistic"] else cr.CR_LINEAR
    return cr.cr_plan_ex(case["L"], case["n"], case["s"], case["m"], case["d"] if d is None else d, model=model,
                         x_dtype=cr.CR_BF16 if case["bf16"] else cr.CR_F32, B=B)


class _Owned:
    """Destroys its plans when the program lets go of them."""

    def __init__(self, *plans):
        self.plans = plans

    def __del__(self):
        torch.cuda.synchronize()
        for plan in self.plans:
            cr.cr_plan_destroy(plan)


def _slab_vectors(plan, d, steps, gen):
    """Gradients of independent row ranges; a slab is the sum over the ranges it covers, so that redundant copies agree."""
    rb, re, _, _ = cr.cr_plan_get_segments(plan)
    cuts = np.unique(np.concatenate([rb, re]))
    stride = (len(rb) * d + 3) // 4 * 4                  # a step's slabs start on a 16-byte boundary
    G = torch.zeros(steps, stride, device="cuda")
    for t in range(steps):
        atoms = torch.randn(len(cuts) - 1, d, generator=gen, device="cuda")
        for q, (lo, hi) in enumerate(zip(np.searchsorted(cuts, rb), np.searchsorted(cuts, re))):
            torch.sum(atoms[lo:hi], dim=0, out=G[t, q * d:(q + 1) * d])
    return G, stride


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = {"case": case, "masks": _masks(case, seed)}
    m, d = case["m"], case["d"]
    if case["kind"] == "layers":
        plans, B = [], None
        for width in LAYERS:                             # the code does not depend on the width: the first plan's serves all
            plans.append(_plan(case, width, B))
            B = cr.cr_plan_get_B(plans[0]) if B is None else B
        state["owned"] = _Owned(*plans)
        state["plans"] = plans
        state["G"] = [_slab_vectors(p, width, 1, gen)[0][0] for p, width in zip(plans, LAYERS)]
        state["g"] = [torch.empty(width, device="cuda") for width in LAYERS]
        state["stream"] = torch.cuda.current_stream().cuda_stream
        return state
    plan = _plan(case)
    state["owned"] = _Owned(plan)
    state["plan"] = plan
    state["workspace"] = ws = cr.Workspace(plan)
    ws.messages().zero_()                                # stragglers never write their rows
    if case["kind"] == "aggregate":
        state["G"], state["stride"] = _slab_vectors(plan, d, case["steps"], gen)
        state["g"] = torch.empty(case["steps"], d, device="cuda")
        return state
    X = torch.empty(m, d, device="cuda", dtype=torch.bfloat16 if case["bf16"] else torch.float32)
    X.normal_(generator=gen)
    w_star = torch.randn(d, generator=gen, device="cuda")
    y = torch.empty(m, device="cuda")
    rows = max(1, (1 << 28) // d)
    for lo in range(0, m, rows):
        y[lo:lo + rows] = X[lo:lo + rows].float() @ w_star
    if case["logistic"]:
        y += 0.1 * torch.randn(m, generator=gen, device="cuda")
        y = (y > 0).float()
        w0 = torch.randn(d, generator=gen, device="cuda") / math.sqrt(d)
    else:
        y += 0.01 * torch.randn(m, generator=gen, device="cuda")
        w0 = torch.randn(d, generator=gen, device="cuda")
    state.update(X=X, y=y, w0=w0, w_star=w_star, g=torch.empty(d, device="cuda"))
    # a twentieth of what gradient descent on such data can take: the run stays where its gradients are well conditioned
    state["lr"] = 0.1 / (m * (1 + math.sqrt(d / m)) ** 2) * (4.0 if case["logistic"] else 1.0)
    if case["measures"]:
        state["metrics"] = torch.empty(case["steps"], 2, device="cuda")
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "layers":
        for plan, G, g in zip(state["plans"], state["G"], state["g"]):
            cr.cr_aggregate_static(plan, G, state["masks"][0], g, state["stream"])
        return state["g"]
    plan = state["plan"]
    if case["kind"] == "aggregate":
        if case["steps"] > 1:
            cr.cr_aggregate_run(plan, state["G"], state["masks"], state["g"], G_step_stride=state["stride"], g_step_stride=case["d"])
            return state["g"]
        cr.cr_load_partial_grads(plan, state["G"])
        cr.cr_encode_tree(plan, state["masks"][0])
        cr.cr_decode_root(plan, state["g"])
        return {"g": state["g"], "messages": state["workspace"].messages()}
    if case["kind"] == "step":
        cr.cr_partial_grads(plan, state["X"], state["y"], state["w0"])
        cr.cr_encode_tree(plan, state["masks"][0])
        cr.cr_decode_root(plan, state["g"])
        return {"g": state["g"], "slabs": state["workspace"].slab_grads(), "messages": state["workspace"].messages()}
    w = state["w0"].clone()
    cr.cr_gd_run(plan, state["X"], state["y"], w, state["g"], state["masks"], state["lr"], state["w_star"] if case["measures"] else None,
                 state.get("metrics"))
    return {"w": w, "g": state["g"], "metrics": state.get("metrics")}


def work(case):
    """Bytes and operations the results cannot do without: every row, target and needed vector read once (a training run: once per
    step), every result written once; two operations per multiply-add."""
    plan = _plan(case, d=8 if case["kind"] in ("aggregate", "layers") else None)
    slabs, workers = cr.cr_plan_info(plan).num_slabs, cr.cr_plan_info(plan).num_workers
    node = cr.cr_plan_get_segments(plan)[3]
    cr.cr_plan_destroy(plan)
    m, d, steps = case["m"], case["d"], case["steps"]
    live = (case["n"] - case["s"]) / case["n"]           # share of the workers of a level that send
    messages = live * workers
    if case["kind"] in ("aggregate", "layers"):
        used = live * len(node)
        return {"bytes": steps * 4 * d * (used + messages + 1), "flops": steps * 2 * d * (used + messages)}
    data = m * d * (2 if case["bf16"] else 4) + 4 * m
    tree = 2 * d * (live * slabs + messages)
    if case["kind"] == "train":
        return {"bytes": steps * (data + 4 * d * 3), "flops": steps * (4 * m * d + tree)}
    return {"bytes": data + 4 * d * (2 + slabs + messages), "flops": 4 * m * d + tree}


def tolerance(case):
    """Everything is accumulated in fp32 over runs of rows and in fp64 across them.  The same results with the rows cut into other
    runs differ by up to 7e-7 (2-norm; slabs of 10^4 rows and more) and 2.8e-6 (largest entry); a vector decoded over two levels of
    the (8,2) code differs from its sum in 64 bits by 5e-7 and 5.2e-6."""
    return {"rel": 3e-6, "max": 2e-5}
