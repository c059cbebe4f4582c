"""Rows with infinities or NaN reach only what they enter: the sums over a
sample that holds such a row and the scores of the element itself."""
import numpy as np
import pytest
import torch

from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def _blobs(n, d, k, seed):
    rng = np.random.default_rng(seed)
    L = rng.integers(0, k, size=n).astype(np.int32)
    return (rng.uniform(-3, 3, size=(k, d))[L] + rng.standard_normal((n, d))).astype(np.float32), L


def _whole(X, L, k, metric, prec):
    """W_hat with every cluster sampled whole."""
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, metric, prec, t=X.shape[0], seed=1)
    native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy()
    res = {x: v.cpu().numpy() if isinstance(v, torch.Tensor) else v for x, v in native.silh_scores(ctx).items()}
    native.silh_destroy(ctx)
    return W, res


@pytest.mark.parametrize("n,d", [(3000, 5), (3000, 12), (3000, 40), (3000, 100), (12_000, 12)])
def test_euclidean_infinite_row_past_the_centre_rows(n, d):
    """An infinite row is at distance infinity from every element: its
    cluster's sums are infinite, not NaN (it is not among the rows that the
    cluster's centre is the mean of), the other clusters' stay as they are."""
    k = 3
    print(f"nonfinite eucl n={n} d={d}", flush=True)
    X, L = _blobs(n, d, k, seed=d)
    bad = int(np.flatnonzero(L == 0)[600])
    ref, _ = _whole(X, L, k, "eucl", "fp32")
    X[bad, 1] = np.inf
    W, res = _whole(X, L, k, "eucl", "fp32")
    ok = np.arange(n) != bad
    assert np.all(W[ok, 0] == np.inf)
    assert np.array_equal(W[ok, 1:], ref[ok, 1:])
    mine = ok & (L == 0)
    assert np.all(res["a"][mine] == np.inf) and np.isfinite(res["b"][mine]).all()
    assert np.isfinite(res["s"][ok & (L != 0)]).all()


@pytest.mark.parametrize("prec,d,first", [("fp32", 20, 3), ("fp32", 200, 3), ("fp32_valu", 20, 3), ("fp32", 20, 700),
                                          ("bf16", 20, 700), ("bf16", 130, 700), ("fp8", 70, 700)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_cosine_row_that_is_not_finite(prec, d, first, value):
    """Such a row's pairs count 0: the other elements' sums are those without
    it, its own are 0 (first: its place among its cluster's sample rows; bf16
    and fp8 round around the mean of the first 256)."""
    n, k = 3000, 3
    print(f"nonfinite cos {prec} d={d} first={first} value={value}", flush=True)
    X, L = _blobs(n, d, k, seed=d)
    bad = int(np.flatnonzero(L == 0)[first])
    ok = np.arange(n) != bad
    ref, _ = _whole(np.ascontiguousarray(X[ok]), np.ascontiguousarray(L[ok]), k, "cos", prec)
    X[bad, 1] = value
    X[bad, 2] = np.inf
    W, res = _whole(X, L, k, "cos", prec)
    # float64 sums over the same rows in another order; float32: a centre moved
    # in its last bit moves an operand by 2^-24
    assert np.all(np.abs(W[ok].astype(np.float64) - ref) <= 2.0 ** -20 * ref)
    assert np.all(W[bad] == 0.0)
    assert res["a"][bad] == 0.0 and res["b"][bad] == 0.0 and res["s"][bad] == 0.0
    assert all(np.isfinite(res[x]).all() for x in "abs") and np.isfinite(res["mean"])
