"""The silhouette work that is measured: whole requests through the Python
binding, over the sizes, metrics and operand types that the framework serves.

A case names the call (`kind`), the data family (`data`), the sizes and the
options.  Kinds:

  scores  a request end to end: silh_sample_init, silh_pps_sample, silh_scores
  sums    the same with silh_weighted_sums (W_hat of every element and
          cluster) and silh_coh_sep on it
  rows    gl-pps-s: Phase 1, then the scores of m uniform row draws
  exact   silh_exact
  sweep   SweepGraph.run: K clusterings of one dataset as one captured graph
          (k = 2 .. K + 1), the graph kept from run to run

Data families:

  blobs   Gaussian blobs with Zipf(1.1) sizes, centres U[-10, 10]^d, standard
          deviations U[0.5, 2]; the labels are the blobs
  dirs    unit rows around k random directions (a cosine of about 0.35 to
          their own), Zipf(1.1) sizes; the labels are the directions
  exp     16 exponential blobs, o_b + Exp(1) per coordinate, o_b ~ U[0, 10]^d;
          the labels are the Voronoi cells of k random rows
  cells   16 Gaussian blobs as `blobs`, the labels the Voronoi cells of k
          random rows (clusters that touch and overlap)
"""
import math

import numpy as np
import torch

from paper_2607_01993_amd import native

DELTA = 0.01


def listed():
    return [
        # the smallest request of the configurations: every kernel is short,
        # launches and round trips count
        dict(name="small", kind="scores", data="blobs", n=2000, d=8, k=4, t=64, metric="eucl", prec="fp32",
             sampler="pps"),
        # the headline request of bench.py
        dict(name="zipf-eucl-bf16", kind="scores", data="blobs", n=1_000_000, d=32, k=16, t=256, metric="eucl",
             prec="bf16", sampler="pps"),
        # the same dataset under Manhattan (bench.py's comparison leg)
        dict(name="zipf-manh-fp32", kind="scores", data="blobs", n=1_000_000, d=32, k=16, t=256, metric="manh",
             prec="fp32", sampler="pps"),
        # one request of the Canberra k-sweep
        dict(name="sweep-canb-fp32", kind="scores", data="exp", n=500_000, d=64, k=64, t=128, metric="canb",
             prec="fp32", sampler="pps"),
        # the directional workload, the largest request of bench.py
        dict(name="dirs-cos-bf16", kind="scores", data="dirs", n=4_000_000, d=128, k=64, t=512, metric="cos",
             prec="bf16", sampler="pps"),
        # fp8 operands on a dataset with odd sizes
        dict(name="dirs-cos-fp8-odd", kind="scores", data="dirs", n=1_000_003, d=100, k=48, t=300, metric="cos",
             prec="fp8", sampler="pps"),
        # long rows
        dict(name="long-eucl-bf16", kind="scores", data="blobs", n=500_000, d=256, k=16, t=256, metric="eucl",
             prec="bf16", sampler="pps"),
        # a request of the serving pool: many touching clusters, the uniform sampler
        dict(name="serve-eucl-bf16-odd", kind="scores", data="cells", n=150_001, d=16, k=100, t=1024, metric="eucl",
             prec="bf16", sampler="uni"),
        # W_hat of every element and cluster, cohesion and separation
        dict(name="sums-eucl-fp32", kind="sums", data="blobs", n=200_000, d=32, k=16, t=256, metric="eucl",
             prec="fp32", sampler="pps"),
        # the subsampled global estimate at eps = delta = 0.01
        dict(name="rows-eucl-bf16", kind="rows", data="blobs", n=1_000_000, d=32, k=16, t=256, metric="eucl",
             prec="bf16", sampler="pps", m=105_967),
        # the exact silhouette
        dict(name="exact-eucl-fp32", kind="exact", data="cells", n=40_000, d=16, k=9, metric="eucl", prec="fp32"),
        # a Euclidean k-sweep as one captured graph
        dict(name="graph-eucl-bf16", kind="sweep", data="exp", n=100_000, d=64, k=16, t=128, metric="eucl",
             prec="bf16", sampler="pps"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the float operations of one coordinate of one pair, as a share of Canberra's,
# the costliest: what a drawn case may cost depends on its metric
_PAIR_COST = {"eucl": 1.0, "cos": 1.0, "manh": 4.0, "canb": 20.0}


def draw(rng):
    kind = rng.choice(["scores"] * 7 + ["sums", "rows", "exact", "sweep"])
    metric = rng.choice(["eucl", "eucl", "cos", "manh", "canb"]) if kind != "sweep" else "eucl"
    d = _log_int(rng, 3, 256)
    if metric in ("eucl", "cos"):
        prec = rng.choice(["bf16", "bf16", "fp32"])
        if metric == "cos" and d >= 64:
            prec = rng.choice(["bf16", "fp8", "fp32"])
        if d > 128 and prec == "fp32":
            prec = "bf16"
    else:
        prec = "fp32"
    data = {"eucl": rng.choice(["blobs", "cells", "exp"]), "cos": "dirs", "manh": rng.choice(["blobs", "cells"]),
            "canb": "exp"}[metric]
    c = dict(kind=kind, data=data, d=d, k=_log_int(rng, 2, 128), metric=metric, prec=prec)
    if kind == "exact":
        c["n"] = _log_int(rng, 1000, 30_000)
        c["k"] = min(c["k"], 40)
        pairs = float(c["n"]) * c["n"]
    else:
        c["n"] = _log_int(rng, 1500, 1_000_000)
        c["t"] = _log_int(rng, 32, 1024)
        c["sampler"] = rng.choice(["pps", "pps", "uni"])
        if kind == "sweep":
            c["n"] = min(c["n"], 100_000)
            c["k"] = rng.randint(4, 16)
            c["t"] = min(c["t"], 256)
        if kind == "rows":
            c["m"] = _log_int(rng, 500, 100_000)
        pairs = float(c["n"]) * min(c["n"], 1.2 * c["k"] * c["t"]) * (c["k"] / 2.0 if kind == "sweep" else 1.0)
    # no dearer than the largest listed case: n shrinks where the product is large
    cost = pairs * d * _PAIR_COST[metric]
    if cost > 2e12:
        c["n"] = max(1500, int(c["n"] * 2e12 / cost)) | 1
    c["k"] = max(2, min(c["k"], c["n"] // 100))
    return c


# ----------------------------------------------------------------------------
# inputs (on the device, from the seed alone)
# ----------------------------------------------------------------------------
def _zipf(n, k):
    w = np.arange(1, k + 1, dtype=np.float64) ** -1.1
    sizes = np.maximum(1, np.floor(n * w / w.sum())).astype(np.int64)
    sizes[0] += n - int(sizes.sum())
    return sizes


def _cells(X, k, g):
    """Voronoi cells of k random rows (Euclidean)."""
    n = X.shape[0]
    C = X[torch.randperm(n, generator=g, device=X.device)[:k]]
    cn = (C * C).sum(dim=1)
    out = torch.empty(n, dtype=torch.int32, device=X.device)
    for r in range(0, n, 1 << 18):
        out[r:r + (1 << 18)] = torch.argmin(cn[None, :] - 2.0 * (X[r:r + (1 << 18)] @ C.T), dim=1).to(torch.int32)
    return out


def _points(case, g):
    n, d, k = case["n"], case["d"], case["k"]
    dev = "cuda"
    if case["data"] == "exp":
        offs = torch.rand((16, d), generator=g, device=dev) * 10.0
        which = torch.randint(0, 16, (n,), generator=g, device=dev)
        return offs[which] + torch.empty((n, d), device=dev).exponential_(1.0, generator=g), None
    nb = 16 if case["data"] == "cells" else k
    lab = torch.repeat_interleave(torch.arange(nb, device=dev), torch.as_tensor(_zipf(n, nb), device=dev))
    lab = lab[torch.randperm(n, generator=g, device=dev)]
    if case["data"] == "dirs":
        mu = torch.randn((nb, d), generator=g, device=dev)
        mu = mu / mu.norm(dim=1, keepdim=True)
        X = torch.randn((n, d), generator=g, device=dev)
        X.add_(mu[lab], alpha=0.37 * math.sqrt(d))
        X.div_(X.norm(dim=1, keepdim=True).clamp_min(1e-30))
    else:
        cen = torch.rand((nb, d), generator=g, device=dev) * 20.0 - 10.0
        sig = torch.rand((nb,), generator=g, device=dev) * 1.5 + 0.5
        X = torch.randn((n, d), generator=g, device=dev)
        X.mul_(sig[lab, None]).add_(cen[lab])
    return X, lab.to(torch.int32)


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * seed + 17)
    X, lab = _points(case, g)
    if case["kind"] == "sweep":
        return X, torch.stack([_cells(X, k, g) for k in _ks(case)]).contiguous()
    return X, lab.contiguous() if case["data"] in ("blobs", "dirs") else _cells(X, case["k"], g)


def _ks(case):
    return list(range(2, case["k"] + 2))


def prepare(case, seed):
    X, L = _inputs(case, seed)
    state = {"case": case, "X": X, "L": L, "seed": seed}
    if case["kind"] == "sweep":
        state["graph"] = native.SweepGraph(X, L, _ks(case), case["metric"], case["prec"], case["sampler"],
                                           t=case["t"], delta=DELTA, seed=seed)
    return state


def run(state):
    c, X, L, seed = state["case"], state["X"], state["L"], state["seed"]
    kind = c["kind"]
    if kind == "sweep":
        res = state["graph"].run()
        return {"means": res["means"], "best": res["best"], "reruns": res["reruns"]}
    if kind == "exact":
        return native.silh_exact(X, L, c["k"], c["metric"], c["prec"])
    if kind == "rows":
        return native.gl_pps_s(X, L, c["k"], c["m"], c["t"], seed, seed + 1, c["metric"], c["prec"], c["sampler"],
                               delta=DELTA)
    ctx = native.silh_sample_init(X, L, c["k"], c["metric"], c["prec"], c["sampler"], t=c["t"], delta=DELTA,
                                  seed=seed)
    S, per_cluster = native.silh_pps_sample(ctx)
    if kind == "sums":
        W = native.silh_weighted_sums(ctx)
        res = {"W": W, **native.silh_coh_sep(ctx, W)}
    else:
        res = native.silh_scores(ctx)
    native.silh_destroy(ctx)
    res["S"], res["per_cluster"] = S, per_cluster
    return res


def work(case):
    """Every element's distances to the sample of its own cluster and of one
    other cluster (its nearest), or of every cluster where W_hat is asked for:
    2 d operations a pair (a contraction).  Bytes: the rows and labels once,
    the outputs once."""
    n, d, k, kind = case["n"], case["d"], case["k"], case["kind"]
    if kind == "exact":
        return {"bytes": 4 * n * d + 16 * n, "flops": 2.0 * n * (2.0 * n / k) * 2 * d}
    per = min(n / k, 1.15 * case["t"])
    if kind == "sweep":
        K = len(_ks(case))
        pairs = sum(2.0 * n * min(n / kk, 1.15 * case["t"]) for kk in _ks(case))
        return {"bytes": 4 * n * d + 4 * n * K, "flops": pairs * 2 * d}
    if kind == "rows":
        m = case["m"]
        return {"bytes": 4 * min(n, m) * d + 4 * n + 12 * m, "flops": 2.0 * min(n, m) * per * 2 * d}
    if kind == "sums":
        return {"bytes": 4 * n * d + 4 * n + 4 * n * k, "flops": n * k * per * 2 * d}
    return {"bytes": 4 * n * d + 16 * n, "flops": 2.0 * n * per * 2 * d}


# ----------------------------------------------------------------------------
# the same in 64 bits, with torch alone
# ----------------------------------------------------------------------------
def _mulhilo(m, c):
    ml, mh = m & 0xFFFF, m >> 16
    hi = (((c * ml) >> 16) + c * mh) >> 16
    return hi, (c * m) & 0xFFFFFFFF


def _bits53(seed, ids, stream):
    """The 53 bits of Philox4x32-10 at counter (id, 0, stream, 0), key = seed."""
    c = [ids & 0xFFFFFFFF, ids >> 32, torch.full_like(ids, stream), torch.zeros_like(ids)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        hi0, lo0 = _mulhilo(0xD2511F53, c[0])
        hi1, lo1 = _mulhilo(0xCD9E8D57, c[2])
        c = [hi1 ^ c[1] ^ k0, lo1, hi0 ^ c[3] ^ k1, lo0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c[0] << 21) | (c[1] >> 11)


def _uniform(seed, ids, stream):
    return _bits53(seed, ids, stream).to(torch.float64) * 2.0 ** -53


def _unit(X):
    return X / X.norm(dim=1, keepdim=True).clamp_min(1e-300)


def _dist(A, B, metric):
    """All distances between the rows of A and of B (float64)."""
    if metric == "cos":
        return (1.0 - _unit(A) @ _unit(B).T).clamp_(0.0, 2.0)
    if metric == "eucl":
        m = B.mean(dim=0) if B.shape[0] else A.mean(dim=0)
        A, B = A - m, B - m
        sq = (A * A).sum(dim=1)[:, None] + (B * B).sum(dim=1)[None, :] - 2.0 * (A @ B.T.contiguous())
        return sq.clamp_(min=0.0).sqrt_()
    acc = torch.zeros((A.shape[0], B.shape[0]), dtype=torch.float64, device=A.device)
    At, Bt = A.T.contiguous(), B.T.contiguous()
    for c in range(A.shape[1]):
        num = torch.sub(At[c][:, None], Bt[c][None, :]).abs_()
        if metric == "canb":
            num /= At[c].abs()[:, None] + Bt[c].abs()[None, :]
            if bool((At[c] == 0).any()) and bool((Bt[c] == 0).any()):
                num.nan_to_num_(nan=0.0)
        acc += num
    return acc


def _sample(X, L, k, metric, t, seed, sampler):
    """Phase 1 (Algorithm 1): ids of the sampled elements by cluster, their
    inclusion probabilities."""
    sizes = torch.bincount(L, minlength=k).tolist()
    order = torch.argsort(L, stable=True)
    out, at = [], 0
    lnterm = math.log(5.0 * k / DELTA)
    for j in range(k):
        ids = order[at:at + sizes[j]]
        at += sizes[j]
        m = sizes[j]
        if m <= t:
            out.append((ids, torch.ones(m, dtype=torch.float64, device=X.device)))
            continue
        if sampler == "uni":
            p = torch.full((m,), min(1.0, t / m), dtype=torch.float64, device=X.device)
            keep = _uniform(seed, ids, 2) < p
        else:
            f0 = ids[_uniform(seed, ids, 0) < min(1.0, (2.0 / m) * lnterm)]
            g = torch.full((m,), 1.0 / m, dtype=torch.float64, device=X.device)
            if f0.numel():
                step = max(1, (1 << 26) // max(1, f0.numel()))
                D = torch.cat([_dist(X[ids[r:r + step]].double(), X[f0].double(), metric)
                               for r in range(0, m, step)])
                w = D.sum(dim=0)
                g = torch.maximum(g, (D[:, w > 0] / w[w > 0]).amax(dim=1)) if bool((w > 0).any()) else g
            p = (t * g).clamp(max=1.0)
            keep = _uniform(seed, ids, 1) < p
        out.append((ids[keep], p[keep]))
    return out, sizes


def _sums(X, rows, sample, metric):
    """W_hat of the given rows (None: all)."""
    n = X.shape[0] if rows is None else rows.shape[0]
    k = len(sample)
    W = torch.zeros((n, k), dtype=torch.float64, device=X.device)
    if metric == "cos":
        # 1 - x.y is linear in y: the sums of the weights and of the weighted unit rows
        tot = torch.stack([(1.0 / p).sum() for _, p in sample])
        V = torch.stack([(_unit(X[ids].double()) / p[:, None]).sum(dim=0) for ids, p in sample])
        for r in range(0, n, 1 << 18):
            x = X[r:r + (1 << 18)] if rows is None else X[rows[r:r + (1 << 18)]]
            W[r:r + (1 << 18)] = tot[None, :] - _unit(x.double()) @ V.T.contiguous()
        return W
    for j, (ids, p) in enumerate(sample):
        for q in range(0, ids.numel(), 4096):
            Y, w = X[ids[q:q + 4096]].double(), 1.0 / p[q:q + 4096]
            step = max(256, (1 << 22) // max(1, Y.shape[0]))
            for r in range(0, n, step):
                x = X[r:r + step] if rows is None else X[rows[r:r + step]]
                W[r:r + step, j] += _dist(x.double(), Y, metric) @ w
    return W


def _scores(W, L, sizes):
    sz = torch.tensor(sizes, dtype=torch.float64, device=W.device)
    own = L.long()[:, None]
    c = sz[own[:, 0]]
    a = torch.where(c > 1, W.gather(1, own)[:, 0] / (c - 1).clamp(min=1), torch.zeros_like(c))
    B = W / sz.clamp(min=1)[None, :]
    B[:, sz == 0] = math.inf
    B.scatter_(1, own, math.inf)
    b = B.amin(dim=1)
    m = torch.maximum(a, b)
    s = torch.where((c > 1) & (m > 0), (b - a) / m, torch.zeros_like(m))
    return a, b, s


def exact(case, seed):
    kind, k, metric = case["kind"], case["k"], case["metric"]
    # the pairs times the coordinates that torch evaluates one after another
    if metric in ("manh", "canb") and case["n"] * min(case["n"], 1.2 * k * case.get("t", case["n"])) * case["d"] > 4e11:
        return None
    X, L = _inputs(case, seed)
    if kind == "sweep":
        means = []
        for i, kk in enumerate(_ks(case)):
            smp, sizes = _sample(X, L[i], kk, metric, case["t"], seed, case["sampler"])
            means.append(float(_scores(_sums(X, None, smp, metric), L[i], sizes)[2].mean()))
        return {"means": np.array(means), "best": int(np.argmax(means)), "reruns": 0}
    if kind == "exact":
        order = torch.argsort(L, stable=True)
        sizes = torch.bincount(L, minlength=k).tolist()
        ids = torch.split(order, sizes)
        smp = [(i, torch.ones(i.numel(), dtype=torch.float64, device=X.device)) for i in ids]
        a, b, s = _scores(_sums(X, None, smp, metric), L, sizes)
        return {"a": a, "b": b, "s": s, "mean": float(s.mean())}
    smp, sizes = _sample(X, L, k, metric, case["t"], seed, case["sampler"])
    if kind == "rows":
        n, m = case["n"], case["m"]
        B = _bits53(seed + 1, torch.arange(m, dtype=torch.int64, device=X.device), 3)
        rows = ((B >> 26) * n + (((B & ((1 << 26) - 1)) * n) >> 26)) >> 27
        a, b, s = _scores(_sums(X, rows, smp, metric), L[rows], sizes)
        return {"a": a, "b": b, "s": s, "mean": float(s.mean()), "rows": rows.to(torch.int32)}
    per = [ids.numel() for ids, _ in smp]
    W = _sums(X, None, smp, metric)
    if kind == "sums":
        sz = np.array(sizes, dtype=np.float64)
        inside = float((sz * (sz - 1) / 2).sum())
        across = float((sz.sum() ** 2 - (sz * sz).sum()) / 2)
        own = torch.arange(k, device=X.device)[None, :] - L.long()[:, None]
        return {"W": W, "coh": 0.5 * float(W[own == 0].sum()) / inside, "sep": float(W[own > 0].sum()) / across,
                "S": sum(per), "per_cluster": np.array(per)}
    a, b, s = _scores(W, L, sizes)
    return {"a": a, "b": b, "s": s, "mean": float(s.mean()), "S": sum(per), "per_cluster": np.array(per)}
