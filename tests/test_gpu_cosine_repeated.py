"""fp8 cosine on clusters of a few rows repeated many times, whose pairs are no
longer clamped one by one, against float64 cosine distances: within what the
operands' rounding can do to the pairs, and never below 0."""
import numpy as np
import pytest

from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,distinct,copies", [(64, 1, 50), (100, 2, 40), (64, 3, 200), (256, 7, 30)])
def test_repeated_rows(d, distinct, copies):
    print(f"cosine fp8 repeated d={d} rows={distinct} x {copies}", flush=True)
    rng = np.random.default_rng(d + distinct)
    rows = rng.standard_normal((distinct, d))
    other = rng.standard_normal((60, d))
    X = np.concatenate([np.repeat(rows, copies, axis=0), other]).astype(np.float32)
    L = np.concatenate([np.zeros(distinct * copies), np.ones(60)]).astype(np.int32)
    order = rng.permutation(X.shape[0])
    X, L = np.ascontiguousarray(X[order]), L[order]
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, 2, "cos", "fp8", t=X.shape[0], seed=1)   # whole clusters, p = 1
    native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    native.silh_destroy(ctx)
    U = X.astype(np.float64)
    U /= np.linalg.norm(U, axis=1)[:, None]
    for j in (0, 1):
        Y = U[L == j]
        ref = (1.0 - U @ Y.T).sum(axis=1)
        mu = Y[:256].mean(axis=0)
        # e4m3: a coordinate moves by up to 2^-4 of itself, a product of two by
        # 2^-3 + 2^-8 of it; |x~.y~| over coordinates is at most |x~| |y~|
        bar = (2.0 ** -3 + 2.0 ** -8) * np.linalg.norm(U - mu, axis=1) * np.linalg.norm(Y - mu, axis=1).sum()
        assert np.all(np.abs(W[:, j] - ref) <= bar + 1e-5 * Y.shape[0])
        assert np.all(W[:, j] >= 0.0)
