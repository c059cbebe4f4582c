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
