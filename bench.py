"""Benchmark of the AGN hot path on one MI355X.

    python bench.py [--steps K] [--warmup W] [--workload NAME] [--no-cpu-baseline]
    python bench.py --mode eval [--workload NAME]     (evaluation only)

One step is one AGN round: lambda local SGD steps of all n workers
(forward, softmax cross-entropy, backward with the fused update) and the
normalize/commit/pull of the n deltas in the round's commit order.  The
value is whole-job throughput in worker-samples per second
(n * lambda * m per round) with inputs resident in HBM.

Printed: one JSON line with the metric, the per-kernel-class breakdown,
the roofline of the dominant kernel class and the CPU oracle timed on a
bounded sample on the host cores.  The timed region replays the captured
round graph; the dominant class's average launch duration comes from HIP
events around each of its launches in an eager pass of the same kernels on
the same stream right after the timed region.

The line also carries "eval": the evaluation of the central variable on a
held-out set of 10,000 rows (the f(t) of the paper's Eq. 4 curves), in
rows per second, with the roofline of its forward products and the
oracle's evaluation timed on the host.  --mode eval runs only that part
(for a profile that holds only the evaluation's kernels).
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

METRIC = "worker-samples/sec per AGN round on 1 MI355X; MFMA util % + commit HBM GB/s"
PEAK_HBM_GBS = 8000.0
PEAK_TFLOPS = {"fp32": 157.3, "bf16": 2516.6}   # dense MFMA peaks of MI355X
SPLIT_TFLOPS = PEAK_TFLOPS["bf16"] / 6           # float32 products done as six bf16 products
STRIP_MIN_GROUPS = 1024                          # (kStripMinGroups of gemm_f32_strip.hip)
CLASSES = ["fwd", "output", "output_dw", "bwd", "dw_first", "commit"]


def class_work(agn, g):
    """Algorithmic work per round of each kernel class as the library
    launches it: ("flop", FLOPs) for classes of matrix products, ("byte",
    bytes) for the bandwidth classes."""
    out = {}
    for c in CLASSES:
        f, b = agn.agn_kernel_class_work(g.ctx, agn.KERNEL_CLASSES[c])
        out[c] = {"flops": f, "bytes": b}
    return out


def class_peak(wl, c):
    """The MFMA rate that bounds a class's products (TFLOP/s): in float32 that
    of the split products, or the float32 MFMA's for the strip kernels and the
    output layer; a class whose layers differ gets the rate of its flops at
    their layers' rates."""
    if wl.dtype != "fp32":
        return PEAK_TFLOPS[wl.dtype]
    if c not in ("fwd", "eval", "bwd", "dw_first"):
        return PEAK_TFLOPS["fp32"]

    def strips(width, other):
        return (wl.m <= 128 and width % 4 == 0 and other % 4 == 0
                and wl.n * -(-width // 64) >= STRIP_MIN_GROUPS)

    d = wl.dims
    if c == "dw_first":
        return PEAK_TFLOPS["fp32"] if strips(d[1], d[0]) else SPLIT_TFLOPS
    if c == "bwd":
        layers = range(1, wl.num_layers if d[-1] > 32 else wl.num_layers - 1)
        macs = [d[l] * d[l + 1] for l in layers]
        cost = [d[l] * d[l + 1] / (PEAK_TFLOPS["fp32"] if strips(d[l], d[l + 1]) else SPLIT_TFLOPS) for l in layers]
        return sum(macs) / sum(cost) if macs else SPLIT_TFLOPS
    return SPLIT_TFLOPS


def round_peak(wl, work):
    """The MFMA rate that bounds a round: its classes' flops at their rates."""
    flops = {c: w["flops"] for c, w in work.items() if w["flops"] > 0}
    return sum(flops.values()) / sum(f / class_peak(wl, c) for c, f in flops.items())


def bound_of(w, peak):
    """A class of matrix products is MFMA-bound when its algorithmic
    intensity reaches the ridge point (peak FLOP/s over peak bytes/s), else
    bound by HBM; classes without products are HBM-bound."""
    if w["flops"] <= 0:
        return "hbm"
    if w["bytes"] <= 0:
        return "mfma"
    ridge = peak * 1e12 / (PEAK_HBM_GBS * 1e9)
    return "mfma" if w["flops"] / w["bytes"] >= ridge else "hbm"


ADAM = (0.9, 0.999, 1e-8)
# commit rule -> (normalize, staleness_scaled)
COMMIT_RULES = {"agn": (True, False), "accumulated": (False, False), "agn_scaled": (True, True),
                "dynsgd": (False, True)}


def host_cores():
    """Cores this process may run on, and the BLAS thread count the oracle's
    products use (set to match the cores)."""
    cores = len(os.sched_getaffinity(0))
    blas = None
    try:
        from threadpoolctl import threadpool_info, threadpool_limits
        threadpool_limits(limits=cores)
        blas = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        pass
    return cores, blas


def cpu_baseline(wl, X, y, orders, budget_s=20.0, adam=None, normalize=True, scaled=False, full=False):
    """The oracle as it stands, on the host cores, timed on a bounded sample
    of the workload: whole rounds while they fit in about budget_s seconds
    (always with full=True, at least one); when one round would take longer,
    the first workers of round 1, each running its lambda local steps, until
    about budget_s seconds have passed (the server's commits, n float32
    vector additions, are under 1% of an oracle round and are left out)."""
    from oracle import AGNOracle
    cores, blas = host_cores()
    o = AGNOracle(wl.dims, wl.n, wl.lam, wl.eta, wl.m, seed=wl.seed, bf16=wl.dtype == "bf16", adam=adam,
                  normalize=normalize, staleness_scaled=scaled)
    Xo = X
    if X.dtype == np.uint16:
        import workloads as W
        Xo = W.f32_from_bf16_bits(X)
    S = wl.N // wl.n
    # one worker's local steps first: they tell whether a whole round fits
    t0 = time.perf_counter()
    o._worker_round(0, Xo, y, S)
    t1 = time.perf_counter() - t0
    per = wl.lam * wl.m
    if full or t1 * wl.n <= budget_s:
        o = AGNOracle(wl.dims, wl.n, wl.lam, wl.eta, wl.m, seed=wl.seed, bf16=wl.dtype == "bf16",
                      adam=adam, normalize=normalize, staleness_scaled=scaled)
        t0 = time.perf_counter()
        rounds = 0
        while True:
            o.round(X, y, orders[rounds % len(orders)])
            rounds += 1
            if time.perf_counter() - t0 >= budget_s:
                break
        dt = time.perf_counter() - t0
        samples = rounds * wl.worker_samples_per_round
        sample = (f"{rounds} full round(s) of {wl.name} ({samples} worker-samples) in {dt:.1f} s, "
                  "float32 storage / float64 accumulation")
    else:
        k, dt = 1, t1
        while k < wl.n and dt + t1 <= budget_s:
            t0 = time.perf_counter()
            o._worker_round(k, Xo, y, S)
            dt += time.perf_counter() - t0
            k += 1
        samples = k * per
        sample = (f"workers 0..{k - 1} of round 1 of {wl.name}, {wl.lam} local steps each ({samples} "
                  f"worker-samples of the round's {wl.worker_samples_per_round}) in {dt:.1f} s; float32 "
                  "storage / float64 accumulation; the commits (under 1% of an oracle round) not timed")
    out = {"value": samples / dt, "unit": "worker-samples/s", "cores": int(cores), "kind": "oracle",
           "sample": sample}
    if blas is not None:
        out["blas_threads"] = int(blas)
    return out


def measure_eval(agn, g, wl, xh, yh, Xh, yh_host, reps=20, cpu=True):
    """Held-out evaluation of the central variable: rows/s over `reps`
    calls (inputs resident in HBM, one stream synchronization at the end),
    the roofline of the forward products (their launches bracketed by HIP
    events in a separate pass), and the oracle's evaluation on the host."""
    import torch
    rows = int(xh.shape[0])
    for _ in range(2):
        g.evaluate(xh, yh)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        agn.agn_evaluate(g.ctx, xh, yh, rows, g.dtype, want_result=False)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / reps
    res = g.evaluate(xh, yh)
    k = agn.KERNEL_CLASSES["eval"]
    agn.agn_set_kernel_timing(g.ctx, k, True)
    kt = 5
    for _ in range(kt):
        agn.agn_evaluate(g.ctx, xh, yh, rows, g.dtype, want_result=False)
    ms, cnt = agn.agn_kernel_timing(g.ctx, k)
    agn.agn_set_kernel_timing(g.ctx, k, False)
    flops, nbytes = agn.agn_kernel_class_work(g.ctx, k)
    per_call_s = ms * 1e-3 / kt
    peak = class_peak(wl, "eval")
    tf = flops / per_call_s / 1e12
    out = {"rows": rows, "rows_per_s": round(rows / dt, 1), "ms_per_eval": round(dt * 1e3, 4),
           "mean_loss": round(res[0], 6), "accuracy": res[1],
           "roofline": {"bound": bound_of({"flops": flops, "bytes": nbytes}, peak),
                        "achieved": round(tf, 3), "peak": round(peak, 1), "unit": "TFLOP/s",
                        "frac": round(tf / peak, 4), "kernel_class": "eval",
                        "launches_per_eval": cnt // kt,
                        "avg_launch_us": round(ms * 1e3 / max(cnt, 1), 2),
                        "algorithmic_per_eval": flops}}
    if cpu:
        from oracle import evaluate
        cores, blas = host_cores()
        # the oracle evaluates the initial model (the library's initial
        # parameters come from the same generator); the cost of an
        # evaluation does not depend on the parameter values
        from oracle import he_normal_init
        params = he_normal_init(wl.dims, wl.seed)
        t0 = time.perf_counter()
        evaluate(params, Xh, yh_host, bf16=wl.dtype == "bf16")
        ct = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(rows / ct, 1), "unit": "rows/s", "cores": int(cores),
                               "kind": "oracle",
                               "sample": f"{rows} held-out rows evaluated once in {ct:.2f} s, at the "
                                         "initial model's parameters"}
        if blas is not None:
            out["cpu_baseline"]["blas_threads"] = int(blas)
    return out


KERNEL_SOURCES = os.path.join(ROOT, "paper_1710_02368_amd", "csrc")
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_{}.json")


def kernel_source_digest():
    """SHA-256 over the library's kernel sources: stored counter readings
    apply only to the kernels they were taken from."""
    import hashlib
    h = hashlib.sha256()
    for f in sorted(os.listdir(KERNEL_SOURCES)):
        h.update(f.encode())
        with open(os.path.join(KERNEL_SOURCES, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def stored_traffic(workload, kernel_class):
    """HBM bytes per launch of a kernel class from the committed rocprofv3
    FETCH_SIZE / WRITE_SIZE passes (scaled by the copy calibration), or None
    when they were taken on other kernel sources or another workload."""
    try:
        with open(TRAFFIC_FILE.format(workload)) as fh:
            t = json.load(fh)
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256") != kernel_source_digest() or t.get("workload") != workload:
        return None
    c = t.get("classes", {}).get(kernel_class)
    return None if c is None else c["hbm_bytes_per_launch"]


def copy_calibration(nbytes=1 << 30, reps=5):
    """A plain device-to-device copy of known size, to scale the FETCH_SIZE and
    WRITE_SIZE counters (run under rocprofv3 --pmc)."""
    import torch
    x = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
    y = torch.empty_like(x)
    for _ in range(reps):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes": nbytes, "reps": reps}))


def copy_ceiling(total_bytes, reps=5):
    """GB/s of a plain device-to-device copy that reads and writes
    total_bytes in all (half each), timed with events on the copy's stream:
    the rate a streaming kernel of that size reaches on this device, beside
    the published 8 TB/s."""
    import torch
    n = max(1 << 20, int(total_bytes) // 8)
    x = torch.empty(n, dtype=torch.float32, device="cuda").fill_(1.0)
    y = torch.empty_like(x)
    for _ in range(2):
        y.copy_(x)
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(reps):
        y.copy_(x)
    stop.record()
    torch.cuda.synchronize()
    gbs = 8.0 * n * reps / (start.elapsed_time(stop) * 1e-3) / 1e9
    del x, y
    torch.cuda.empty_cache()
    return gbs


# rocprofv3 kernel names -> the kernel classes the library times
def traffic_class(name):
    if "commit_kernel" in name:
        return "commit"
    if "head_dw_kernel" in name:
        return "output_dw"
    if "head_kernel" in name or "softmax_ce" in name:
        return "output"
    if "_bwd_kernel" in name:
        return "bwd"
    if "_dw_kernel" in name or "<false, false, 3>" in name or ", false, false, 3," in name:
        return "dw_first"
    if "<true, true" in name or ", true, true, " in name or "_fwd_kernel" in name or "_fwd8_kernel" in name or "gemm_bf16_dl_big_kernel" in name:
        return "fwd"
    return None


def summarize_traffic(d, workload):
    """FETCH_SIZE / WRITE_SIZE counter passes (rocprofv3 --pmc, csv output,
    under d/{bench,copy}_{FETCH_SIZE,WRITE_SIZE}/) -> HBM bytes per launch
    of each kernel class, scaled by what the same counter reads for the
    1 GiB copy of --copy-calibration; written to profiles/traffic_<workload>.json with
    the digest of the kernel sources, and printed as a text summary."""
    import collections
    import csv

    def rows(sub, counter):
        with open(os.path.join(d, sub, "run_counter_collection.csv")) as fh:
            return [r for r in csv.DictReader(fh) if r["Counter_Name"] == counter]

    def factor(counter):
        vals = [float(r["Counter_Value"]) for r in rows(f"copy_{counter}", counter)
                if "copy" in r["Kernel_Name"].lower() or "elementwise" in r["Kernel_Name"].lower()]
        kib = max(v for v in vals if v > 0)
        return (1 << 30) / (kib * 1024.0), kib

    out = {"workload": workload, "kernel_source_sha256": kernel_source_digest(), "classes": {}}
    lines = []
    per = {}
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        f, kib = factor(counter)
        lines.append(f"copy calibration (1 GiB device copy): {counter} {kib:.0f} KiB -> factor {f:.4f}")
        cls, kern = collections.defaultdict(list), collections.defaultdict(list)
        for r in rows(f"bench_{counter}", counter):
            v = float(r["Counter_Value"]) * 1024 * f
            kern[r["Kernel_Name"][:90]].append(v)
            c = traffic_class(r["Kernel_Name"])
            if c:
                cls[c].append(v)
        per[counter] = (cls, kern)
    fcls, fkern = per["FETCH_SIZE"]
    wcls, wkern = per["WRITE_SIZE"]
    for c in sorted(fcls):
        f = sum(fcls[c]) / len(fcls[c])
        w = sum(wcls.get(c, [0.0])) / max(1, len(wcls.get(c, [0.0])))
        out["classes"][c] = {"hbm_bytes_per_launch": f + w, "fetch_bytes_per_launch": f,
                             "write_bytes_per_launch": w, "launches_sampled": len(fcls[c])}
        lines.append(f"class {c:9s}: fetch {f / 1e6:9.2f} MB + write {w / 1e6:9.2f} MB per launch "
                     f"({len(fcls[c])} launches)")
    for k in sorted(fkern):
        f = sum(fkern[k]) / len(fkern[k])
        w = sum(wkern.get(k, [0.0])) / max(1, len(wkern.get(k, [0.0])))
        lines.append(f"  {k[:80]:80s} fetch {f / 1e6:9.2f} MB write {w / 1e6:9.2f} MB")
    with open(TRAFFIC_FILE.format(workload), "w") as fh:
        json.dump(out, fh, indent=1)
    print("\n".join(lines))


MFMA_FILE = os.path.join(ROOT, "profiles", "mfma_{}.json")


def summarize_mfma(d, workload, dtype):
    """MFMA counter pass (rocprofv3 --pmc MfmaUtil MfmaFlopsF32 MfmaFlopsBF16
    GRBM_GUI_ACTIVE for float32 workloads, without MfmaFlopsF32 for bf16 ones,
    csv output under d/; a float32 product done as six bf16 products counts
    as a sixth of its bf16 flops) -> per kernel class: the MFMA busy
    fraction (MfmaUtil: busy cycles of the matrix units over the dispatch's
    active cycles times the SIMD count, averaged over the class's launches
    weighted by their durations) and the MFMA flops the counters saw per
    launch (with the achieved rate over the launches' durations); written to profiles/mfma_<workload>.json with the digest of the
    kernel sources, and printed as a text summary."""
    import collections
    import csv
    weights = {"MfmaFlopsBF16": 1.0} if dtype == "bf16" else {"MfmaFlopsF32": 1.0, "MfmaFlopsBF16": 1.0 / 6}
    flops_name = "MfmaFlopsBF16" if dtype == "bf16" else "MfmaFlopsF32 + MfmaFlopsBF16 / 6"
    per = collections.defaultdict(dict)
    names, dur = {}, {}
    with open(os.path.join(d, "run_counter_collection.csv")) as fh:
        for r in csv.DictReader(fh):
            k = r["Dispatch_Id"]
            per[k][r["Counter_Name"]] = per[k].get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
            names[k] = r["Kernel_Name"]
            dur[k] = (float(r["End_Timestamp"]) - float(r["Start_Timestamp"])) * 1e-9
    cls = collections.defaultdict(lambda: {"busy_w": 0.0, "active": 0.0, "flops": 0.0, "launches": 0})
    kern = collections.defaultdict(lambda: {"busy_w": 0.0, "active": 0.0, "flops": 0.0, "launches": 0})
    for k, v in per.items():
        if "MfmaUtil" not in v or dur[k] <= 0:
            continue
        for key, table in ((traffic_class(names[k]), cls), (names[k][:90], kern)):
            if key is None:
                continue
            e = table[key]
            e["busy_w"] += v["MfmaUtil"] / 100.0 * dur[k]
            e["active"] += dur[k]
            e["flops"] += sum(w * v.get(name, 0.0) for name, w in weights.items())
            e["launches"] += 1
    out = {"workload": workload, "kernel_source_sha256": kernel_source_digest(), "counter_flops": flops_name,
           "classes": {}}
    lines = [f"MFMA counters ({flops_name}, MfmaUtil = SQ_VALU_MFMA_BUSY_CYCLES / (GRBM_GUI_ACTIVE x SIMDs))"]
    for c in sorted(cls):
        e = cls[c]
        if e["active"] <= 0:
            continue
        util = e["busy_w"] / e["active"]
        fl = e["flops"] / e["launches"]
        rate = e["flops"] / e["active"] / 1e12
        out["classes"][c] = {"mfma_busy": util, "mfma_flops_per_launch": fl, "counter_tflops": rate,
                             "launches_sampled": e["launches"]}
        lines.append(f"class {c:9s}: MFMA busy {100 * util:6.2f} %   MFMA flops per launch {fl / 1e9:10.3f} G "
                     f"= {rate:7.2f} TFLOP/s over the launches' durations ({e['launches']} launches)")
    for k in sorted(kern, key=lambda k: -kern[k]["active"]):
        e = kern[k]
        if e["active"] <= 0:
            continue
        lines.append(f"  {k[:80]:80s} busy {100 * e['busy_w'] / e['active']:6.2f} %  "
                     f"{e['flops'] / e['launches'] / 1e9:9.3f} GFLOP/launch  ({e['launches']})")
    with open(MFMA_FILE.format(workload), "w") as fh:
        json.dump(out, fh, indent=1)
    print("\n".join(lines))


def stored_mfma(workload, kernel_class):
    """The MFMA busy fraction of a kernel class from the committed counter
    pass, or None when it was taken on other kernel sources."""
    try:
        with open(MFMA_FILE.format(workload)) as fh:
            t = json.load(fh)
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256") != kernel_source_digest():
        return None
    c = t.get("classes", {}).get(kernel_class)
    return None if c is None else round(c["mfma_busy"], 4)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="mlp2000_n40")
    ap.add_argument("--optimizer", choices=["sgd", "adam"], default="sgd",
                    help="local rule: plain SGD (the paper's Eq. 1) or Adam (beta 0.9/0.999, eps 1e-8)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-eval", action="store_true",
                    help="skip the held-out evaluation (counter passes of the round's kernels alone)")
    ap.add_argument("--cpu-budget", type=float, default=20.0)
    ap.add_argument("--cpu-full-round", action="store_true",
                    help="time the oracle over at least one whole round, however long it takes")
    ap.add_argument("--commit", choices=sorted(COMMIT_RULES), default="agn",
                    help="commit rule: agn (a / lambda, the default), accumulated (a), or either scaled by "
                         "1 / (staleness + 1) (agn_scaled, dynsgd)")
    ap.add_argument("--mode", choices=["round", "eval"], default="round",
                    help="round: the AGN round (default line, with the evaluation); eval: evaluation only")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a 1 GiB device copy (counter calibration)")
    ap.add_argument("--summarize-mfma", metavar="DIR",
                    help="turn the MFMA counter pass under DIR into profiles/mfma_<workload>.json "
                         "for --workload (no GPU needed)")
    ap.add_argument("--summarize-traffic", metavar="DIR",
                    help="turn the FETCH_SIZE / WRITE_SIZE counter passes under DIR into "
                         "profiles/traffic_<workload>.json (no GPU needed)")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration()
        return
    if args.summarize_traffic:
        summarize_traffic(args.summarize_traffic, args.workload)
        return
    if args.summarize_mfma:
        import workloads as W
        summarize_mfma(args.summarize_mfma, args.workload, W.workload(args.workload).dtype)
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}); the multi-GPU "
              "sharding of the commit is a design, not a build", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_1710_02368_amd as agn
    import workloads as W

    assert torch.cuda.is_available(), "bench.py needs a ROCm GPU"
    wl = W.workload(args.workload)
    X, y = W.make_data(wl)
    orders = W.commit_orders(wl, rounds=max(wl.rounds, 1))
    xd = torch.from_numpy(X.view(np.int16) if X.dtype == np.uint16 else X).cuda()
    yd = torch.from_numpy(y).cuda()
    adam = ADAM if args.optimizer == "adam" else None
    normalize, scaled = COMMIT_RULES[args.commit]
    g = agn.AGN(wl.dims, wl.n, wl.lam, wl.eta, wl.m, seed=wl.seed, dtype=wl.dtype, adam=adam,
                normalize=normalize, staleness_scaled=scaled)
    order_at = lambda i: orders[i % len(orders)]
    Xh, yh = W.make_heldout(wl)
    xh = torch.from_numpy(Xh.view(np.int16) if Xh.dtype == np.uint16 else Xh).cuda()
    yh_d = torch.from_numpy(yh).cuda()

    if args.mode == "eval":
        ev = measure_eval(agn, g, wl, xh, yh_d, Xh, yh, reps=max(args.steps, 1),
                          cpu=not args.no_cpu_baseline)
        out = {"metric": "held-out rows/sec evaluated (central variable, forward + loss + argmax)",
               "value": ev["rows_per_s"], "unit": "rows/s", "n_gpus": 1, "steps": max(args.steps, 1),
               "warmup": 2, "ms_per_step": ev["ms_per_eval"], "higher_is_better": True, "scaling": "weak",
               "vs_baseline": None, "dtype": "f32" if wl.dtype == "fp32" else "bf16", "data": "synthetic",
               "config": {"workload": wl.name + "_heldout", "dims": list(wl.dims), "rows": ev["rows"]},
               "roofline": dict(ev["roofline"], traffic=None)}
        if "cpu_baseline" in ev:
            out["cpu_baseline"] = ev["cpu_baseline"]
        g.close()
        print(json.dumps(out), flush=True)
        return

    for i in range(args.warmup):
        g.round(xd, yd, order_at(i))
    torch.cuda.synchronize()

    # per-class breakdown (untimed pass, every class bracketed by events)
    for c in CLASSES:
        agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES[c], True)
    prof_rounds = 2
    for i in range(prof_rounds):
        g.round(xd, yd, order_at(i))
    work = class_work(agn, g)
    breakdown = {}
    for c in CLASSES:
        ms, cnt = agn.agn_kernel_timing(g.ctx, agn.KERNEL_CLASSES[c])
        agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES[c], False)
        if cnt == 0:
            continue
        per_round_s = ms * 1e-3 / prof_rounds
        e = {"ms_per_round": round(per_round_s * 1e3, 4), "launches_per_round": cnt // prof_rounds}
        if work[c]["flops"] > 0:
            e["TFLOP/s"] = round(work[c]["flops"] / per_round_s / 1e12, 2)
            e["mfma_frac"] = round(work[c]["flops"] / per_round_s / 1e12 / class_peak(wl, c), 4)
        if work[c]["bytes"] > 0:
            e["GB/s"] = round(work[c]["bytes"] / per_round_s / 1e9, 1)
            e["hbm_frac"] = round(work[c]["bytes"] / per_round_s / 1e9 / PEAK_HBM_GBS, 4)
        breakdown[c] = e
    dominant = max(breakdown, key=lambda c: breakdown[c]["ms_per_round"])

    # timed region: K rounds, replaying the captured round graph (the product path)
    for i in range(2):
        g.round(xd, yd, order_at(i))     # (re)capture outside the timed region
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        g.round(xd, yd, order_at(args.warmup + i))
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0

    # kernel timing pass right after it: the same kernels launched eagerly on
    # the same stream, each launch of the dominant class between HIP events
    kt_rounds = max(1, min(args.steps, 10))
    agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES[dominant], True)
    for i in range(kt_rounds):
        g.round(xd, yd, order_at(i))
    dom_ms, dom_cnt = agn.agn_kernel_timing(g.ctx, agn.KERNEL_CLASSES[dominant])
    agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES[dominant], False)

    # commit kernel alone (HBM roofline of the normalize/commit/pull)
    agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES["commit"], True)
    for i in range(5):
        g.round(xd, yd, order_at(i))
    c_ms, c_cnt = agn.agn_kernel_timing(g.ctx, agn.KERNEL_CLASSES["commit"])
    agn.agn_set_kernel_timing(g.ctx, agn.KERNEL_CLASSES["commit"], False)
    torch.cuda.synchronize()

    # evaluation of the trained central variable on the held-out set
    ev = None if args.no_eval else measure_eval(agn, g, wl, xh, yh_d, Xh, yh, cpu=not args.no_cpu_baseline)

    value = args.steps * wl.worker_samples_per_round / dt
    wd = work[dominant]
    peak = class_peak(wl, dominant)
    bound = bound_of(wd, peak)
    launches_per_round = max(dom_cnt, 1) / kt_rounds
    avg_s = dom_ms * 1e-3 / max(dom_cnt, 1)
    if bound == "mfma":
        per_launch = wd["flops"] / launches_per_round
        achieved = per_launch / avg_s / 1e12
        roof = {"bound": "mfma", "achieved": round(achieved, 3), "peak": round(peak, 1),
                "unit": "TFLOP/s", "frac": round(achieved / peak, 4)}
    else:
        per_launch = wd["bytes"] / launches_per_round
        achieved = per_launch / avg_s / 1e9
        roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": round(achieved / PEAK_HBM_GBS, 4)}
    roof.update({"traffic": stored_traffic(wl.name, dominant), "counter_mfma_busy": stored_mfma(wl.name, dominant),
                 "kernel_class": dominant,
                 "avg_launch_us": round(avg_s * 1e6, 2), "algorithmic_per_launch": per_launch,
                 "launches": dom_cnt})
    c_avg = c_ms * 1e-3 / max(c_cnt, 1)
    commit_gbs = work["commit"]["bytes"] / c_avg / 1e9
    copy_gbs = copy_ceiling(work["commit"]["bytes"])
    out = {
        "metric": METRIC, "value": round(value, 1), "unit": "worker-samples/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(dt * 1e3 / args.steps, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32" if wl.dtype == "fp32" else "bf16", "data": "synthetic",
        "config": {"workload": wl.name, "optimizer": args.optimizer, "commit": args.commit,
                   "dims": list(wl.dims), "n": wl.n, "lambda": wl.lam, "m": wl.m,
                   "eta": wl.eta, "commit_order": wl.order, "num_samples": wl.N,
                   "worker_samples_per_round": wl.worker_samples_per_round},
        "roofline": roof,
        "commit_roofline": {"bound": "hbm", "achieved": round(commit_gbs, 1), "peak": PEAK_HBM_GBS,
                            "unit": "GB/s", "frac": round(commit_gbs / PEAK_HBM_GBS, 4),
                            "avg_launch_us": round(c_avg * 1e6, 2),
                            "algorithmic_per_launch": work["commit"]["bytes"],
                            "traffic": stored_traffic(wl.name, "commit"),
                            "copy_ceiling": {"achieved": round(copy_gbs, 1), "unit": "GB/s",
                                             "kind": "device-to-device copy of the same bytes, same run"},
                            "frac_of_copy": round(commit_gbs / copy_gbs, 4)},
        "round_mfma_util": round(wl.flops_per_round / (dt / args.steps) / 1e12 / round_peak(wl, work), 4),
        "kernels": breakdown,
    }
    if ev is not None:
        out["eval"] = ev
    g.close()
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(wl, X, y, orders, budget_s=args.cpu_budget, adam=adam,
                                           normalize=normalize, scaled=scaled, full=args.cpu_full_round)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
