#!/usr/bin/env python3
"""Benchmark of the CodedReduce hot path on one MI355X.

One "step" is one pass of the whole path over one batch of synthetic input already resident in HBM:
host-drawn straggler mask -> cr_partial_grads -> cr_encode_tree -> cr_decode_root -> gradient step
(issued through cr_gd_run -- cr_aggregate_run for the aggregation-only workloads -- which enqueues these steps for every mask;
the gradient step rides in the launch of the decode, and that in the encode's where the vectors are short).

Prints ONE JSON line, short enough to be kept whole.  Its top level is the headline workload (configuration 5: the largest,
end-to-end iterations/s); "configs" holds for every benchmark configuration and for the comparison workloads of the paper's
computation-load discussion, all measured in this run: iterations/s, the median time of the dominant kernel (HIP events on the
library's stream over the timed steps), the fraction of its roofline, the CPU oracle timed on a bounded sample of the same workload,
and the parity of one GPU iteration with that oracle.  --detail FILE writes the whole records (every kernel with average, minimum,
median and maximum, the work split, the samples) there as JSON.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME] [--detail FILE]

roofline.frac is the fraction of the resource that binds: for the memory-bound kernels the bytes HBM really moved per
launch (rocprofv3 FETCH_SIZE + WRITE_SIZE of the same kernel and work split, profiles/hbm_traffic.json) over the
kernel's time, against 8 TB/s; needed_GBps counts the bytes that the kernel's arithmetic cannot do without (the data once where the
holders' common sums are formed once, once per holder where every holder does its own).  What stage 1 takes when every holder does
its own arithmetic is stage1_every_holder_ms.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0            # MI355X published HBM3E bandwidth
FP32_VECTOR_PEAK_TFLOPS = 78.6    # 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz x 2 flop; the published 157.3 counts packed instructions
KERNEL_NAMES = ["partial_grads", "reduce_pieces", "encode", "decode", "update"]
DESCRIPTIONS = {
    "cfg1": "CR tree L=2 n=3 s=1, linear regression fp32, m=1200 d=100",
    "cfg2": "CR tree L=2 n=4 s=1 (20 workers), linear regression fp32, m=100000 d=10000, GD lr=1e-6, random mask per step",
    "cfg3": "CR tree L=3 n=4 s=1 (84 workers), logistic regression fp32, m=252000 d=4096, random mask per step",
    "cfg4": "aggregation only: CR tree L=2 n=8 s=2 (72 workers), 248 fp32 partition-gradient vectors of length 2^24, encode+decode",
    "cfg5": "CR tree L=3 n=6 s=2 (258 workers), linear regression, X bf16 / fp32 accumulate, m=2064000 d=1024, random mask per step",
    "gc20": "one-layer gradient coding, n=20 s=4 (same data and resiliency as cfg2), linear regression fp32, m=100000 d=10000",
    "umw20": "uncoded master-worker, n=20 s=0 (same data as cfg2), linear regression fp32, m=100000 d=10000",
    "paper84": "the paper's linear-regression experiment: CR tree L=3 n=4 s=1 (84 workers), fp32, m=7644 d=6500, noise N(0,1)",
    "nn12": "aggregation only: CR tree L=2 n=12 s=5 (156 workers, resiliency 5/12), fp32 partition-gradient vectors of length 117706 (network sized), encode+decode",
}
HEADLINE = "cfg5"
DEFAULT_SET = ["cfg5", "cfg2", "gc20", "umw20", "cfg3", "cfg4", "cfg1", "nn12", "paper84"]     # cfg2, gc20, umw20 share one data set


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


SPLITS = ["equal_ranges", "row_cells", "shared_cells", "rows_once"]


def split_signature(info) -> str:
    """What identifies the kernel and work split a traffic record belongs to."""
    kind = SPLITS[info.split_kind] if info.split_kind >= 0 else "none"
    return f"{kind}:{info.split_value}:team{info.stage1_team_size}x{info.stage1_teams_per_group}:staged{info.stage1_staged}"


def load_traffic(workload: str, signature: str, algorithmic=None):
    """HBM bytes per launch of the dominant kernel from the committed rocprofv3 --pmc summary, if it was taken with this kernel
    and work split (else None and the reason).  algorithmic: this run's algorithmic bytes per launch, where they depend on how its
    steps divide into calls (a call of several masks writes the messages of the last ones only): the record is scaled to them."""
    path = os.path.join(ROOT, "profiles", "hbm_traffic.json")
    if not os.path.exists(path):
        return None, "no traffic record"
    with open(path) as f:
        entry = json.load(f).get(workload)
    if entry is None:
        return None, "no traffic record for this workload"
    if entry.get("split_signature") not in (None, signature):
        return None, f"traffic record is for {entry.get('split_signature')}, this run uses {signature}"
    traffic = entry.get("bytes_per_launch")
    if traffic and algorithmic and entry.get("algorithmic_bytes_per_launch"):
        traffic = round(traffic * algorithmic / entry["algorithmic_bytes_per_launch"])
    return traffic, entry.get("source")


def stats(ms: np.ndarray) -> dict:
    return {"avg": float(ms.mean()), "min": float(ms.min()), "median": float(np.median(ms)), "max": float(ms.max())}


def cpu_baseline_regression(cfg, data, w_host, mask, g_gpu, budget_s: float):
    """The oracle as it stands: the CR tree literally (every holder visits its own rows) in fp64 on the host cores."""
    from oracle import cr_tree, gc_code, native

    L, n, s = cfg["L"], cfg["n"], cfg["s"]
    B = gc_code.design_code(n, s, L, 190201981)[0]
    own, _ = cr_tree.cr_allocate(L, n, s, cfg["m"], B)
    slabs = cr_tree.slabs_of(own)
    visits = sum(e - b for _, b, e, _ in slabs)
    native.num_threads()
    t0 = time.perf_counter()
    done_rows = 0
    node_grads = [np.zeros(cfg["d"]) for _ in own]
    complete = True
    for k, (node, b, e, c) in enumerate(slabs):
        node_grads[node] += float(c) * native.segment_gradient(data["X"], data["y"], w_host, b, e, cfg["model"])
        done_rows += e - b
        if time.perf_counter() - t0 > budget_s and k + 1 < len(slabs):
            complete = False
            break
    parity = None
    if complete:
        rows = {}
        _, g = cr_tree.cr_execute(L, n, s, node_grads, mask, lambda T: rows.setdefault(T, gc_code.decoding_row(B, T)))
        parity = float(np.linalg.norm(g_gpu - g) / np.linalg.norm(g))
    elapsed = time.perf_counter() - t0
    its = (done_rows / visits) / elapsed
    sample = (f"one whole CR iteration ({visits} row visits, all {len(slabs)} slabs, tree execute included)" if complete else
              f"first {k + 1} of {len(slabs)} slabs ({done_rows} of {visits} row visits), scaled to one iteration")
    return {"value": its, "unit": "iterations/s", "cores": native.num_threads(), "kind": "oracle", "sample": sample,
            "seconds": elapsed}, parity


def cpu_baseline_aggregation(cfg, slabs_host_cols, cols, mask, g_gpu_cols, d):
    """The oracle's tree execution (numpy fp64, one thread) on a sample of columns of the caller-supplied slab gradients."""
    from oracle import cr_tree, gc_code

    L, n, s = cfg["L"], cfg["n"], cfg["s"]
    B = gc_code.design_code(n, s, L, 190201981)[0]
    own, _ = cr_tree.cr_allocate(L, n, s, cfg["m"], B)
    slabs = cr_tree.slabs_of(own)
    t0 = time.perf_counter()
    ng = [np.zeros(len(cols)) for _ in own]
    for q, (node, _, _, c) in enumerate(slabs):
        ng[node] += float(c) * slabs_host_cols[q].astype(np.float64)
    rows = {}
    _, g = cr_tree.cr_execute(L, n, s, ng, mask, lambda T: rows.setdefault(T, gc_code.decoding_row(B, T)))
    elapsed = time.perf_counter() - t0
    parity = float(np.linalg.norm(g_gpu_cols - g) / np.linalg.norm(g))
    return {"value": (len(cols) / d) / elapsed, "unit": "iterations/s", "cores": 1, "kind": "oracle",
            "sample": f"{len(cols)} of {d} columns of one encode+decode (all {len(slabs)} slabs, every message), scaled to one iteration",
            "seconds": elapsed}, parity


def every_holder_ms(cfg, X_dev, y_dev, w_dev) -> float:
    """Stage-1 milliseconds (median of 5 launches) when every holder of a row does its own arithmetic on it (row cells): what the
    redundancy of the scheme costs, where the default split forms the holders' common sums once."""
    import paper_1902_01981_amd as cr

    plan = cr.cr_plan_ex(cfg["L"], cfg["n"], cfg["s"], cfg["m"], cfg["d"], model=cfg["model"], x_dtype=cfg["x_dtype"])
    row_bytes = cfg["d"] * (2 if cfg["x_dtype"] else 4)
    visits = cr.cr_plan_info(plan).row_visits
    cell = min(min(512, max(96, ((2 << 20) // row_bytes + 16) // 32 * 32)), max(16, (visits // 2048 + 15) // 16 * 16))
    cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROW_CELLS, cell)
    ws = cr.Workspace(plan)
    cr.cr_partial_grads(plan, X_dev, y_dev, w_dev)
    cr.cr_profile_enable(plan, 1 << cr.CR_K_PARTIAL_GRADS)
    for _ in range(5):
        cr.cr_partial_grads(plan, X_dev, y_dev, w_dev)
    ms = float(np.median(cr.cr_profile_samples(plan, cr.CR_K_PARTIAL_GRADS)))
    cr.cr_plan_destroy(plan)
    del ws
    return ms


_DATA_CACHE = {}


def dataset(cfg, wl):
    key = (cfg["seed"], cfg["m"], cfg["d"], cfg["x_dtype"], cfg["model"], cfg["noise"], cfg["w0_std"])
    if key not in _DATA_CACHE:
        _DATA_CACHE.clear()                             # one data set in host memory at a time
        _DATA_CACHE[key] = wl.make_dataset(cfg, threads=min(16, os.cpu_count() or 8))
    return _DATA_CACHE[key]


def run_workload(name: str, steps: int, warmup: int, cpu_budget: float, args) -> dict:
    import torch

    import paper_1902_01981_amd as cr
    from cr_inputs import workloads as wl

    cfg = wl.config(name)
    L, n, s, m, d = cfg["L"], cfg["n"], cfg["s"], cfg["m"], cfg["d"]
    aggregate = cfg["model"] == wl.AGGREGATE_ONLY
    t0 = time.perf_counter()
    plan = cr.cr_plan_ex(L, n, s, m, d, model=cfg["model"], x_dtype=cfg["x_dtype"])
    if not aggregate:
        if args.teams:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_EQUAL_RANGES, args.teams)
        elif args.cell_rows:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_ROW_CELLS, args.cell_rows)
        elif args.shared_rows:
            cr.cr_plan_set_split(plan, cr.CR_SPLIT_SHARED_CELLS, args.shared_rows)

    # ---- inputs, generated on the host from the seed and moved to HBM before any timing
    data = None
    if aggregate:
        rb, re_, coef, node = cr.cr_plan_get_segments(plan)
        cuts, member = wl.atoms_of(rb, re_)
        atoms_dev = torch.empty((len(cuts) - 1, d), dtype=torch.float32, device="cuda")
        step_cols = 1 << 22
        for lo in range(0, d, step_cols):
            hi = min(d, lo + step_cols)
            atoms_dev[:, lo:hi] = torch.from_numpy(wl.atom_vectors(cfg["seed"], len(cuts) - 1, lo, hi)).cuda()
        G_dev = torch.empty((len(member), d), dtype=torch.float32, device="cuda")
        for q, idx in enumerate(member):                 # input preparation: redundant copies of a row range must agree
            G_dev[q] = atoms_dev[idx].sum(dim=0)
        del atoms_dev
        w_dev = torch.zeros(d, dtype=torch.float32, device="cuda")
    else:
        data = dataset(cfg, wl)
        X = data["X"]
        X_dev = torch.from_numpy(X.view(np.int16) if X.dtype == np.uint16 else X).cuda()
        y_dev = torch.from_numpy(data["y"]).cuda()
        w_dev = torch.from_numpy(data["w0"]).cuda()
    log(f"{name}: inputs ready in {time.perf_counter() - t0:.1f}s")
    ws = cr.Workspace(plan)
    info = ws.info
    g_dev = torch.empty(d, dtype=torch.float32, device="cuda")
    rng = wl.mask_stream(cfg)
    lr = float(cfg["lr"])

    def draw(count):
        return np.stack([wl.draw_mask(rng, L, n, s) for _ in range(count)])

    def run(masks):
        # the whole path for every host-drawn straggler mask; for regression workloads the gradient-descent loop is one library
        # call per batch of masks, which enqueues its steps without waiting for the device
        for lo in range(0, len(masks), 16):
            if aggregate:
                cr.cr_aggregate_run(plan, G_dev, masks[lo:lo + 16], g_dev)
            else:
                cr.cr_gd_run(plan, X_dev, y_dev, w_dev, g_dev, masks[lo:lo + 16], lr)

    dominant = "encode" if aggregate else "partial_grads"
    dom_id = KERNEL_NAMES.index(dominant)

    def read_kernels(into):
        for kid, kname in enumerate(KERNEL_NAMES):
            ms, launches, nbytes = cr.cr_profile_read(plan, kid)
            if launches:
                into[kname] = {"ms": stats(cr.cr_profile_samples(plan, kid)), "launches": launches,
                               "algorithmic_bytes_per_launch": nbytes // launches,
                               "algorithmic_GBps": nbytes / (ms * 1e-3) / 1e9 if ms > 0 else None}

    # Clock ramp, untimed and before the warm-up steps: after the idle stretch in which the inputs were generated the device
    # takes about 10 ms of continuous load to reach its running clocks (the first launches of a burst run up to 40 % slower,
    # see the per-launch samples), so the path is run until it has kept the device busy for RAMP_MS.  Then the W warm-up steps,
    # the synchronisation, and exactly K timed steps whose masks are already drawn (no host work between the two).
    ramp_steps = 0
    probe_masks = draw(4)
    t_r = time.perf_counter()
    run(probe_masks)
    torch.cuda.synchronize()
    per_step = max((time.perf_counter() - t_r) / 4, 1e-6)
    ramp_steps = int(min(2000, max(0, args.ramp_ms * 1e-3 / per_step)))
    if ramp_steps:
        run(draw(ramp_steps))
    run(draw(warmup))
    timed_masks = draw(steps)
    extra_masks = draw(min(steps, 10))
    torch.cuda.synchronize()
    # timed region: only the dominant kernel is bracketed by events (every bracket costs a few microseconds of device time)
    cr.cr_profile_enable(plan, 1 << dom_id)
    torch.cuda.synchronize()
    t_start = time.perf_counter()
    run(timed_masks)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t_start
    kernels = {}
    read_kernels(kernels)
    if aggregate and kernels[dominant]["launches"] < steps:
        # one launch for up to 16 masks (the batches of run()): figures per mask
        masks_of = np.array([min(16, steps - lo) for lo in range(0, steps, 16)], dtype=np.float64)
        ms = cr.cr_profile_samples(plan, dom_id).astype(np.float64)
        kernels[dominant].update(ms=dict(stats(ms / masks_of), avg=float(ms.sum() / steps)), masks_per_launch=masks_of.tolist(),
                                 algorithmic_bytes_per_launch=kernels[dominant]["algorithmic_bytes_per_launch"] * len(ms) // steps)
    # the other kernels, from a few more steps outside the timed region with every launch bracketed
    cr.cr_profile_enable(plan, True)
    run(extra_masks)
    others = {}
    read_kernels(others)
    for kname, entry in others.items():
        kernels.setdefault(kname, dict(entry, timed_region=False))
    cr.cr_profile_enable(plan, False)
    dk = kernels[dominant]
    avg_s = dk["ms"]["avg"] * 1e-3
    signature = split_signature(info) if not aggregate else "encode"
    traffic, traffic_source = load_traffic(name, signature, dk["algorithmic_bytes_per_launch"] if aggregate else None)
    holder_ms = every_holder_ms(cfg, X_dev, y_dev, w_dev) if not aggregate and s > 0 else None
    # yardstick: what a plain streaming read of the same buffer reaches on this device right now
    big = G_dev if aggregate else X_dev
    sink = torch.empty(16384, dtype=torch.float32, device="cuda")
    nbytes = min(big.numel() * big.element_size(), 4 << 30) // 16 * 16
    stream_gbps = cr.cr_probe_read_bandwidth(big, nbytes, sink, 10, torch.cuda.current_stream().cuda_stream) if nbytes >= (1 << 20) else None
    traffic_gbps = traffic / avg_s / 1e9 if traffic else None
    hbm = {"traffic": traffic, "traffic_source": traffic_source, "traffic_GBps": traffic_gbps,
           "traffic_frac_of_peak": traffic_gbps / HBM_PEAK_GBPS if traffic else None,
           "frac_of_stream_read": traffic_gbps / stream_gbps if traffic and stream_gbps else None,
           "traffic_frac_whole_step": traffic / (elapsed / steps) / 1e9 / HBM_PEAK_GBPS if traffic else None,
           "stream_read_GBps": stream_gbps}
    every_holder = not aggregate and s > 0 and info.split_kind in (cr.CR_SPLIT_EQUAL_RANGES, cr.CR_SPLIT_ROW_CELLS)
    if aggregate or every_holder:
        needed = dk["algorithmic_bytes_per_launch"]
    else:
        needed = m * d * (2 if cfg["x_dtype"] == wl.BF16 else 4) + 4 * m + 4 * d * (info.num_slabs + 1)
        dk.pop("algorithmic_bytes_per_launch")           # these charge every holder's read of a row
        dk.pop("algorithmic_GBps")
    common = {"kernel": dominant, "kernel_ms": dk["ms"], "needed_bytes_per_launch": needed, "needed_GBps": needed / avg_s / 1e9}
    if every_holder and cfg["x_dtype"] == wl.BF16:
        # bf16 rows, every holder's arithmetic done separately (--teams, --cell-rows): stage 1 is bound by vector-ALU issue (a widening operation and two multiply-adds per element), not by memory:
        # 4 flop per element of X visited, against the vector peak of the instructions this build issues
        flops = 4.0 * info.row_visits * d
        achieved = flops / avg_s / 1e12
        roofline = dict(common, bound="alu", achieved=achieved, peak=FP32_VECTOR_PEAK_TFLOPS, unit="TFLOP/s",
                        frac=achieved / FP32_VECTOR_PEAK_TFLOPS, traffic=traffic, flops_per_launch=flops,
                        peak_derivation="256 compute units x 4 SIMDs x 16 lanes x 2.4 GHz x 2 flop per multiply-add = 78.6 TFLOP/s; "
                                        "the published 157.3 TFLOP/s counts packed fp32 instructions, which this build does not issue",
                        # the least this instruction set allows: no instruction multiplies a bf16 operand by an fp32 one, so an
                        # element costs a widening operation and two multiply-adds = three vector instructions of 4 clocks per
                        # wavefront; frac_of_issue_floor = that time / the measured time
                        issue_floor_ms=3.0 * info.row_visits * d / 64.0 * 4.0 / (256 * 4 * 2.4e9) * 1e3,
                        frac_of_issue_floor=3.0 * info.row_visits * d / 64.0 * 4.0 / (256 * 4 * 2.4e9) / avg_s,
                        hbm_view=hbm)
    else:
        roofline = dict(common, bound="hbm", achieved=traffic_gbps, peak=HBM_PEAK_GBPS, unit="GB/s",
                        frac=traffic_gbps / HBM_PEAK_GBPS if traffic else None, **hbm)

    # ---- CPU baseline: the oracle on the host cores, same inputs, bounded; also a parity check of one more GPU iteration
    baseline, parity = None, None
    if cpu_budget > 0:
        mask = wl.draw_mask(rng, L, n, s)
        if aggregate:
            ncols = int(min(d, max(4096, (1 << 18) * cpu_budget / 20.0))) // 4 * 4
            cols = np.arange(ncols) + ((d - ncols) // 2) // 4 * 4          # a block in the middle of the vectors
            cr.cr_load_partial_grads(plan, G_dev)
            cr.cr_encode_tree(plan, mask)
            cr.cr_decode_root(plan, g_dev)
            cr.cr_synchronize(plan)
            baseline, parity = cpu_baseline_aggregation(cfg, G_dev[:, cols[0]:cols[-1] + 1].cpu().numpy(), cols, mask,
                                                        g_dev[cols[0]:cols[-1] + 1].cpu().numpy().astype(np.float64), d)
        else:
            # at the starting model: after many steps w sits at the optimum, where the gradient is the difference of large
            # cancelling terms and a relative error says nothing
            w_host = data["w0"]
            w_dev.copy_(torch.from_numpy(w_host))
            cr.cr_partial_grads(plan, X_dev, y_dev, w_dev)
            cr.cr_encode_tree(plan, mask)
            cr.cr_decode_root(plan, g_dev)
            cr.cr_synchronize(plan)
            baseline, parity = cpu_baseline_regression(cfg, data, w_host, mask, g_dev.cpu().numpy().astype(np.float64), cpu_budget)
        log(f"{name}: cpu baseline {baseline}, parity {parity}")

    out = {
        "workload": f"{name}: {DESCRIPTIONS[name]}",
        "value": steps / elapsed,
        "unit": "iterations/s",
        "steps": steps,
        "warmup": warmup,
        "clock_ramp_steps": ramp_steps + 4,
        "ms_per_step": elapsed / steps * 1e3,
        "us_per_iteration": elapsed / steps * 1e6,
        "dtype": "f32",          # the arithmetic type: bf16 rows are widened; products are fp32, sums over rows fp32 or fp64
        "config": {"workload": f"{name}: {DESCRIPTIONS[name]}", "L": L, "n": n, "s": s, "m": m, "d": d,
                   "x_storage": "bf16" if cfg["x_dtype"] == wl.BF16 else "f32",
                   "workers": info.num_workers, "slabs": info.num_slabs, "row_visits": info.row_visits,
                   "computation_load": info.r_cr, "rows_per_worker": [info.min_rows, info.max_rows],
                   "stage1_teams": info.num_teams, "stage1_pieces": info.num_pieces, "code_gamma": info.gamma,
                   "stage1_split": SPLITS[info.split_kind] if info.split_kind >= 0 else None,
                   "stage1_split_value": info.split_value,
                   "stage1_arithmetic": None if aggregate else "every holder" if every_holder
                   else "every slab range once" if info.split_value == cr.CR_ROWS_WHOLE_RANGES else "every row once, for all its holders",
                   "stage1_every_holder_ms": holder_ms, "stage1_team_size": info.stage1_team_size,
                   "stage1_holders_per_workgroup": info.stage1_teams_per_group if info.stage1_staged else 1,
                   "l2_domains": info.l2_domains, "l2_sharing_checked": info.l2_sharing, "split_signature": signature},
        "roofline": roofline,
        "kernels": kernels,
        "cpu_baseline": baseline,
        "parity_rel_l2_vs_oracle": parity,
    }
    cr.cr_plan_destroy(plan)
    del ws, big
    if aggregate:
        del G_dev
    else:
        del X_dev, y_dev
    torch.cuda.empty_cache()
    return out


def rounded(v):
    """The record with its measured numbers to six digits."""
    if isinstance(v, dict):
        return {k: rounded(x) for k, x in v.items()}
    return float(f"{v:.6g}") if isinstance(v, float) else v


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default=None, choices=sorted(DESCRIPTIONS),
                    help="run this workload only (default: configuration 5 as the headline and every other one under 'configs')")
    ap.add_argument("--cpu-budget", type=float, default=12.0, help="seconds of oracle work per workload for the CPU baseline (0 = skip)")
    ap.add_argument("--ramp-ms", type=float, default=60.0,
                    help="untimed load before the warm-up steps, in milliseconds of device time, to bring the clocks up (0 = none)")
    ap.add_argument("--teams", type=int, default=0, help="stage-1 split: this many equal contiguous ranges")
    ap.add_argument("--cell-rows", type=int, default=0, help="stage-1 split: row cells of this many rows")
    ap.add_argument("--shared-rows", type=int, default=0, help="stage-1 split: shared cells of at most this many rows")
    ap.add_argument("--detail", default=None, help="write the whole records to this file")
    ap.add_argument("--calibrate", action="store_true",
                    help="run only a plain 1 GiB elementwise copy kernel a few times (reference for rocprofv3 byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        return 2

    import torch

    import paper_1902_01981_amd as cr

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 1
    if args.calibrate:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(5):
            torch.mul(src, 1.0, out=dst)                 # reads 2^30 bytes, writes 2^30 bytes per launch
        torch.cuda.synchronize()
        print(json.dumps({"calibrate": "torch.mul(src, 1.0, out=dst)", "bytes_read": 1 << 30, "bytes_written": 1 << 30, "launches": 5}))
        return 0
    cr.load_library()
    names = [args.workload] if args.workload else DEFAULT_SET
    records = {}
    for name in names:
        records[name] = run_workload(name, args.steps, args.warmup, args.cpu_budget, args)
        log(f"{name}: {records[name]['value']:.1f} it/s, dominant kernel {records[name]['roofline']['kernel_ms']}")
    if args.detail:
        with open(args.detail, "w") as f:
            json.dump(records, f, indent=1)
    head = records[names[0]]
    roof, cpu = head["roofline"], head["cpu_baseline"]
    out = {
        "metric": "CR gradient iterations/sec",
        "value": head["value"],
        "unit": "iterations/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": head["dtype"],
        "data": "synthetic",
        "config": {k: head["config"][k] for k in ("workload", "x_storage", "workers", "stage1_split", "stage1_arithmetic", "stage1_every_holder_ms")},
        "roofline": {"kernel": roof["kernel"], "kernel_ms": roof["kernel_ms"]["median"],
                     **{k: roof.get(k) for k in ("bound", "achieved", "peak", "unit", "frac", "traffic", "needed_GBps", "stream_read_GBps")}},
        "cpu_baseline": cpu and {k: cpu[k] for k in ("value", "unit", "cores", "kind", "sample")},
        "parity_rel_l2_vs_oracle": head["parity_rel_l2_vs_oracle"],
    }
    if len(names) > 1:
        out["configs"] = {k: {"value": v["value"], "kernel_ms": v["roofline"]["kernel_ms"]["median"], "frac": v["roofline"]["frac"],
                              "cpu": v["cpu_baseline"] and v["cpu_baseline"]["value"], "parity": v["parity_rel_l2_vs_oracle"]} for k, v in records.items()}
        # Section III-C's comparison of computation loads on configuration 2's data (20 workers, one straggler in four tolerated):
        # uncoded master-worker (r = 1/N), CodedReduce on the (4,2) tree (r_CR), gradient coding ((S+1)/N)
        out["computation_load_comparison"] = {
            k: {"load_r": records[k]["config"]["computation_load"], "stage1_ms": records[k]["roofline"]["kernel_ms"]["median"],
                "every_holder_ms": records[k]["config"]["stage1_every_holder_ms"]} for k in ("umw20", "cfg2", "gc20") if k in records}
    out = rounded(out)
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
