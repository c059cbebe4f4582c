"""The margin of the Euclidean bounds covers the largest rounding of bf16
operands: a cluster that only the rounding makes the nearest is not left out."""
import numpy as np
import pytest

from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m1,m2", [(19, 75), (18, 71), (40, 158)])
def test_rounding_decides_the_nearest(m1, m2):
    """Three clusters of equal rows: 0, 257 on m1 coordinates (256 in bf16) and
    128.51 on the other m2 (129 in bf16).  Exactly, the third is nearer to the
    first; with the operands' rounding the second is.  Nine more lie far off, so
    that the bounds pay."""
    m, d, k = 2000, m1 + m2, 12
    print(f"bounds margin d={d}", flush=True)
    X = np.zeros((k * m, d), dtype=np.float32)
    X[m:2 * m, :m1] = 257.0
    X[2 * m:3 * m, m1:] = 128.51
    for j in range(3, k):
        X[j * m:(j + 1) * m, j] = 1024.0 * j
    L = np.repeat(np.arange(k, dtype=np.int32), m)
    order = np.random.default_rng(d).permutation(k * m)
    X, L = np.ascontiguousarray(X[order]), L[order]
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "eucl", "bf16", t=m, seed=1)   # whole clusters, p = 1
    native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    b = native.silh_scores(ctx)["b"].cpu().numpy()
    native.silh_destroy(ctx)
    first = L == 0
    assert np.all(W[first, 1] < W[first, 2])      # the case at hand
    B = np.where(np.arange(k)[None, :] == L[:, None], np.inf, W / m)
    assert np.all(np.abs(b - B.min(axis=1)) <= 2.0 ** -22 * b)   # one more rounding to float32
