"""Phase-2 measurements on each workload shape, beside the least time that the
memory allows.

    python -m paper_2607_01993_amd.configs [--out FILE] [--only zipf,d256] [--metrics canb,manh]

Workloads (seeded, synthetic):
  small       n = 2,000, d = 8, k = 4 Gaussian blobs, t = 64
  zipf        n = 1e6, d = 32, k = 16 Zipf Gaussian blobs, t = 256
  directional n = 4e6, d = 128, k = 64 vMF blobs (kappa 50), t = 512, cosine
  sweep-k64   n = 5e5, d = 64 exponential blobs, Voronoi k = 64, t = 128
  d256        n = 5e5, d = 256, k = 16 Zipf Gaussian blobs, t = 256

For every (workload, metric, operands) Phase 2 (bounds, tables and records
included) is timed with HIP events (median of 5 requests after one warm-up).
pairs_per_s counts all n*S pairs as answered, also those that the Euclidean
bounds, the cosine records and the Manhattan / Canberra tables save the
kernels, so no rate of the arithmetic units is derived from it; the roofline
is of the bytes that Phase 2 cannot do without.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import statistics
import sys

HBM_GBS = 8000.0  # published peak of one MI355X


def phase2_kernel(metric, prec, d):
    """The kernel that Phase 2 spends its time in on these workloads."""
    if metric == "cos":
        return "k_p2_cos"
    if metric == "eucl":
        if prec == "bf16" or (prec == "fp32" and d <= 128):
            return "k_p2_mfma"
        return "k_p2_valu" if d <= 128 else "k_p2_valu_wide"
    return "k_tab_eval"


def phase2_floor(metric, prec, n, d, outputs, ms):
    """Roofline of Phase 2 by its least traffic: the rows, the labels and
    `outputs` float32 arrays of n once, over the time of Phase 2.  What bounds
    the kernels themselves (square roots and sums, dot products, table
    searches) depends on the data and is not counted here."""
    least = n * (4.0 * d + 4.0 + 4.0 * outputs)
    ach = least / (ms * 1e-3) / 1e9
    return {"bound": "hbm", "achieved": ach, "peak": HBM_GBS, "unit": "GB/s", "frac": ach / HBM_GBS,
            "work": f"{least:.0f} bytes: rows, labels and {outputs} outputs once",
            "kernel": phase2_kernel(metric, prec, d), "kernel_ms": ms}


def log(msg):
    print(f"# {msg}", file=sys.stderr, flush=True)


def measure(native, X, L, k, metric, prec, t, reps=5):
    times, S = [], 0
    for i in range(reps + 1):
        ctx = native.silh_sample_init(X, L, k, metric, prec, "pps", t=t, seed=1)
        native.silh_prof_enable(ctx, 2)
        S, _ = native.silh_pps_sample(ctx)
        native.silh_scores(ctx, a=False, b=False, s=False, mean=True)
        ms = native.silh_prof_get(ctx)["phase2"][1]
        native.silh_destroy(ctx)
        if i > 0:
            times.append(ms)
    ms = statistics.median(times)
    n, d = X.shape
    pairs = float(n) * S / (ms * 1e-3)
    out = {"metric": metric, "prec": prec, "n": n, "d": d, "k": k, "t": t, "S": S, "phase2_ms": ms,
           "pairs_per_s": pairs}
    out["roofline"] = phase2_floor(metric, prec, n, d, 0, ms)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--out", default=None)
    ap.add_argument("--skip-directional", action="store_true")
    ap.add_argument("--only", default=None, help="comma-separated workloads (small, zipf, sweep-k64, d256, directional)")
    ap.add_argument("--metrics", default=None, help="comma-separated metrics to measure (default: all)")
    args = ap.parse_args()
    only = set(args.only.split(",")) if args.only else None
    mets = set(args.metrics.split(",")) if args.metrics else None

    def want(workload, metric=None):
        return (only is None or workload in only) and (metric is None or mets is None or metric in mets)
    import torch

    from . import native, synth

    def dev(X, L):
        return torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda()

    rows = []
    if want("small"):
        X, L = dev(*synth.config_small())
        for metric, prec in (("eucl", "fp32"), ("eucl", "bf16")):
            if want("small", metric):
                rows.append({"workload": "small", **measure(native, X, L, 4, metric, prec, 64)})
    if want("zipf"):
        X, L = dev(*synth.config_zipf_gauss())
        for metric, prec in (("eucl", "bf16"), ("eucl", "fp32"), ("cos", "bf16"), ("manh", "fp32"), ("canb", "fp32")):
            if want("zipf", metric):
                rows.append({"workload": "zipf", **measure(native, X, L, 16, metric, prec, 256)})
        log("zipf done")
        del X, L
    if want("sweep-k64"):
        Xe = synth.config_sweep()
        cen = synth.voronoi_centers(Xe.shape[0], 64, (3, 64))
        Le = synth.voronoi_labels(Xe, cen)
        X, L = dev(Xe, Le)
        for metric, prec in (("eucl", "bf16"), ("canb", "fp32")):
            if want("sweep-k64", metric):
                rows.append({"workload": "sweep-k64", **measure(native, X, L, 64, metric, prec, 128)})
        log("sweep-k64 done")
    if want("d256"):
        n = 500_000
        Xg, Lg = synth.gaussian_blobs(n, 256, 16, seed=9, sizes=synth.zipf_sizes(n, 16), sigma=(0.5, 2.0))
        X, L = dev(Xg, Lg)
        for metric, prec in (("eucl", "bf16"), ("cos", "fp8"), ("manh", "fp32")):
            if want("d256", metric):
                rows.append({"workload": "d256", **measure(native, X, L, 16, metric, prec, 256, reps=3)})
        log("d256 done")
        del X, L
    if not args.skip_directional and want("directional", "cos"):
        Xv, Lv = synth.config_vmf_cos()
        log("directional data ready")
        X, L = dev(Xv, Lv)
        del Xv, Lv
        for prec in ("bf16", "fp8", "fp32"):
            rows.append({"workload": "directional", **measure(native, X, L, 64, "cos", prec, 512, reps=3)})
            log(f"directional {prec} done")
    line = json.dumps({"phase2_by_workload": rows})
    print(line, flush=True)
    if args.out:
        with open(args.out, "w") as f:
            f.write(line + "\n")


if __name__ == "__main__":
    main()
