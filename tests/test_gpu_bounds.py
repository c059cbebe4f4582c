"""Euclidean scores through the cluster bounds (only the clusters an element
can need are evaluated) against the sums of every cluster (silh_weighted_sums):
a_hat is the own cluster's sum and b_hat the smallest of the others', also
where clusters touch, coincide, are empty or have an empty sample."""
import numpy as np
import pytest

from parity_util import dev
from paper_2607_01993_amd import native, synth

pytestmark = pytest.mark.gpu


def _data(kind, n, d, k, seed):
    rng = np.random.default_rng(seed)
    if kind == "blobs":
        return synth.gaussian_blobs(n, d, k, seed=seed, sizes=synth.zipf_sizes(n, k), sigma=(0.5, 2.0))
    if kind == "cells":
        X = synth.exp_blobs(n, d, 5, seed=seed)
        return X, synth.voronoi_labels(X, synth.voronoi_centers(n, k, (seed, k)))
    if kind == "same":      # every cluster drawn from one blob, far from the origin; one label unused
        X = (1000.0 + rng.standard_normal((n, d))).astype(np.float32)
        return X, rng.integers(0, k - 1, size=n).astype(np.int32)
    X, L = synth.split_blobs(n, d, k, seed=seed, dup=1e-4)
    return X, L


@pytest.mark.parametrize("kind,n,d,k,t,prec,sampler", [
    ("blobs", 50_001, 5, 3, 256, "fp32", "pps"), ("blobs", 40_031, 33, 16, 128, "bf16", "pps"),
    ("cells", 30_000, 16, 129, 8, "bf16", "uni"), ("cells", 20_000, 64, 65, 16, "fp32", "pps"),
    ("cells", 16_001, 100, 33, 64, "bf16", "pps"), ("same", 20_000, 8, 20, 64, "bf16", "pps"),
    ("same", 20_000, 40, 7, 200, "fp32", "uni"), ("split", 24_000, 24, 4, 300, "fp32", "pps"),
    ("split", 24_000, 200, 5, 300, "bf16", "pps"), ("cells", 60_000, 12, 200, 2, "bf16", "uni")])
def test_scores_equal_the_smallest_sums(kind, n, d, k, t, prec, sampler):
    print(f"bounds {kind} n={n} d={d} k={k} t={t} {prec} {sampler}", flush=True)
    X, L = _data(kind, n, d, k, seed=n % 97)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "eucl", prec, sampler, t=t, seed=5)
    S, per = native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    res = {x: v.cpu().numpy().astype(np.float64) if x != "mean" else v for x, v in native.silh_scores(ctx).items()}
    native.silh_destroy(ctx)
    assert n * S >= 1 << 24     # the bounds are in use
    sizes = np.bincount(L, minlength=k).astype(np.float64)
    rows = np.arange(n)
    a = np.where(sizes[L] > 1, W[rows, L] / np.maximum(sizes[L] - 1, 1), 0.0)
    B = W / np.maximum(sizes, 1)[None, :]
    B[:, sizes == 0] = np.inf
    B[rows, L] = np.inf
    b = B.min(axis=1)
    # both sides round the same float64 sums once to float32
    assert np.all(np.abs(res["a"] - a) <= 2.0 ** -22 * a)
    assert np.all(np.abs(res["b"] - b) <= 2.0 ** -22 * b)
    m = np.maximum(a, b)
    s = np.where((sizes[L] > 1) & (m > 0), (b - a) / np.where(m > 0, m, 1.0), 0.0)
    assert np.max(np.abs(res["s"] - s)) <= 2.0 ** -20
    assert abs(res["mean"] - s.mean()) <= 2.0 ** -20
