"""Manhattan and Canberra sums by per-coordinate tables (n >= 1024) against
float64 sums over the pairs: values of both signs, zeros, duplicates, constant
coordinates, tight clusters, values outside the tables' range (summed
directly), clusters of more rows than one table holds, elements far outside
the sample."""
import numpy as np
import pytest

import oracle
from oracle.distance import dist_matrix
from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def _data(kind, n, d, k, seed):
    rng = np.random.default_rng(seed)
    L = rng.integers(0, k, size=n).astype(np.int32)
    c = rng.uniform(-3, 3, size=(k, d))
    if kind == "gauss":
        X = c[L] + rng.standard_normal((n, d))
        X[rng.random((n, d)) < 0.1] = 0.0
    elif kind == "pos":
        X = np.abs(c)[L] + rng.exponential(1.0, size=(n, d))
        X[:40] *= 50.0                       # elements far beyond the sample
        X[40:60] *= 1e-5
    elif kind == "tight":
        X = 5.0 + c[L] + 1e-4 * rng.standard_normal((n, d))
        X[L == 0] = X[L == 0][:1]            # one cluster of identical points
    elif kind == "int":
        X = rng.poisson(1.5, size=(n, d)).astype(float)
        X[:, 0] = 2.0                        # a constant coordinate
        X[:, 1 % d] *= -1.0
    else:
        X = rng.lognormal(0.0, 8.0, size=(n, d)) * rng.choice([-1.0, 1.0], size=(n, d))
    return np.ascontiguousarray(X.astype(np.float32)), L


@pytest.mark.parametrize("metric", ["manh", "canb"])
@pytest.mark.parametrize("kind,n,d,k,t", [("gauss", 8192, 3, 4, 100), ("gauss", 9001, 33, 7, 64),
                                          ("pos", 20_000, 17, 16, 130), ("pos", 8192, 200, 3, 300),
                                          ("tight", 9000, 12, 5, 200), ("int", 12_345, 9, 6, 256),
                                          ("wide", 8200, 5, 3, 90), ("gauss", 9999, 6, 3, 9999),
                                          ("pos", 300_000, 4, 2, 48), ("gauss", 1024, 1, 2, 16),
                                          ("int", 2500, 64, 40, 60), ("wide", 1100, 256, 2, 600)])
def test_sums_equal_the_pairs(metric, kind, n, d, k, t):
    print(f"tables {metric} {kind} n={n} d={d} k={k} t={t}", flush=True)
    X, L = _data(kind, n, d, k, seed=n % 89)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, metric, "fp32", t=t, seed=3)
    S, per = native.silh_pps_sample(ctx)
    view = native.silh_sample_view(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    res = native.silh_scores(ctx)
    native.silh_destroy(ctx)
    rows = np.unique(np.concatenate([np.arange(64), np.random.default_rng(1).integers(0, n, 400),
                                     view["gid"][:: max(1, S // 200)]]))
    ref = np.zeros((rows.size, k))
    for j in range(k):
        F = view["gid"][view["offsets"][j]:view["offsets"][j + 1]]
        ref[:, j] = (dist_matrix(X[rows], X[F], metric) / view["p"][F][None, :]).sum(axis=1)
    # each table's value to 2^-22 of itself (an ulp of its ends, the weights'
    # rounding, the cubic), one rounding of the result; direct sums of 32 rows
    # in float32: 2^-20 covers both
    assert np.all(np.abs(W[rows] - ref) <= 2.0 ** -20 * ref), np.max(np.abs(W[rows] - ref) / np.maximum(ref, 1e-300))
    est = oracle.silhouette.scores_from_weights(W, L, np.bincount(L, minlength=k))
    for x, v in zip("abs", est):
        assert np.max(np.abs(res[x].cpu().numpy() - v) - 2.0 ** -21 * np.abs(v)) <= (2.0 ** -20 if x == "s" else 0.0), x
    assert abs(res["mean"] - est[2].mean()) <= 2.0 ** -20
