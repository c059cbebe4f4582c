"""Manhattan and Canberra tables over the values they take: whole datasets of
small magnitude (neighbouring knots 10^-14 and less apart), columns of zeros,
and what Canberra's tables refuse (summed directly, two rows with one
reciprocal) and Manhattan's take."""
import numpy as np
import pytest

from oracle.distance import dist_matrix
from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def sums_and_pairs(X, L, k, metric, t, seed=3, count=300):
    """W_hat of 2 count elements, sampled ones among them, and the same from the
    pairs in float64."""
    n = X.shape[0]
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, metric, "fp32", t=t, seed=seed)
    S, _ = native.silh_pps_sample(ctx)
    view = native.silh_sample_view(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    res = native.silh_scores(ctx)
    native.silh_destroy(ctx)
    rows = np.unique(np.concatenate([np.random.default_rng(1).integers(0, n, count), view["gid"][:: max(1, S // count)]]))
    ref = np.zeros((rows.size, k))
    for j in range(k):
        F = view["gid"][view["offsets"][j]:view["offsets"][j + 1]]
        ref[:, j] = (dist_matrix(X[rows], X[F], metric) / view["p"][F][None, :]).sum(axis=1)
    return W, res, rows, ref


@pytest.mark.parametrize("metric", ["manh", "canb"])
@pytest.mark.parametrize("scale", [1e-6, 1e-7, 1.5e-8, 2e-9])
def test_small_magnitudes(metric, scale):
    n, d, k, t = 600_000, 24, 2, 600
    print(f"tables small {metric} scale={scale}", flush=True)
    rng = np.random.default_rng(5)
    X = ((0.6 + rng.exponential(1.0, size=(n, d))) * scale).astype(np.float32)   # all above 2^-30
    L = rng.integers(0, k, size=n).astype(np.int32)
    W, res, rows, ref = sums_and_pairs(X, L, k, metric, t)
    assert np.isfinite(W).all() and np.isfinite(res["mean"])
    assert np.isfinite(res["a"].cpu().numpy()).all() and np.isfinite(res["s"].cpu().numpy()).all()
    # a table's value to 2^-22 of itself (an ulp of its ends, the weights'
    # rounding, the cubic), one rounding of the result
    assert np.all(np.abs(W[rows] - ref) <= 2.0 ** -20 * ref), np.max(np.abs(W[rows] - ref) / ref)


@pytest.mark.parametrize("zeros", [0.5, 0.99, 1.0])
def test_sparse_canberra(zeros):
    """Columns of zeros: an element's zero meets a sampled zero at distance
    exactly 0, also where nearly the whole sample is 0."""
    n, d, k, t = 30_000, 9, 3, 700
    print(f"tables sparse zeros={zeros}", flush=True)
    rng = np.random.default_rng(7)
    X = rng.exponential(1.0, size=(n, d)) * rng.choice([-1.0, 1.0], size=(n, d))
    L = rng.integers(0, k, size=n).astype(np.int32)
    X[rng.random((n, d)) < zeros] = 0.0
    X[L == 0] = 0.0                      # one cluster of zero rows only
    W, res, rows, ref = sums_and_pairs(X.astype(np.float32), L, k, "canb", t)
    assert np.all(W[L == 0, 0] == 0.0)
    assert np.all(res["a"].cpu().numpy()[L == 0] == 0.0)
    if zeros == 1.0:                     # every distance is 0
        assert np.all(W == 0.0) and res["mean"] == 0.0 and np.all(res["s"].cpu().numpy() == 0.0)
    # as above
    assert np.all(np.abs(W[rows] - ref) <= 2.0 ** -20 * ref), np.max(np.abs(W[rows] - ref) / np.maximum(ref, 1e-300))


@pytest.mark.parametrize("metric", ["manh", "canb"])
@pytest.mark.parametrize("kind", ["1e-12", "1e11", "1e-41", "1e16", "1e36", "mixed", "lognormal"])
@pytest.mark.parametrize("n,d,k,t", [(5001, 7, 3, 131), (200_003, 4, 16, 40)])
def test_any_magnitude(metric, kind, n, d, k, t):
    if metric == "canb" and kind == "1e-41":
        pytest.skip("a sum of two subnormal magnitudes is taken as the smallest normal number (the 0/0 guard)")
    print(f"tables range {metric} {kind} n={n}", flush=True)
    rng = np.random.default_rng(n)
    L = rng.integers(0, k, size=n).astype(np.int32)
    X = 1.0 + rng.exponential(1.0, size=(n, d))
    if kind == "mixed":                    # a column in the range, others below, above and with zeros
        X *= np.array([1.0, 1e-13, 1e12, 1e18, 1.0, 1e-25, 1e12])[None, :d]
        X[rng.random((n, d)) < 0.05] = 0.0
        X *= rng.choice([-1.0, 1.0], size=(n, d))
    elif kind == "lognormal":
        X = np.exp(8.0 * rng.standard_normal((n, d)))
    else:
        X *= float(kind)
    W, res, rows, ref = sums_and_pairs(X.astype(np.float32), L, k, metric, t)
    # as above; summed directly 32 terms in float32, each good to 2^-22
    with np.errstate(over="ignore"):
        ok = ref < 3e38                    # (1e36: sums past the float32 range)
    assert np.all(np.abs(W[rows] - ref)[ok] <= 2.0 ** -19 * ref[ok]), np.max(np.abs(W[rows] - ref)[ok] / ref[ok])
    assert np.all(np.isinf(W[rows][~ok]))
