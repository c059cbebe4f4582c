"""Phase 1's W pass where one work item's initial-sample rows go to several
blocks, or to one block in several rounds (more than 24 rows at d > 64, more
than 64 below), against the float64 oracle: ids exactly, W and p to 1e-13."""
import numpy as np
import pytest

import oracle
from paper_2607_01993_amd import native, synth
from parity_util import assert_same_sets, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric,n,d,k,delta", [
    ("eucl", 2500, 8, 3, 1e-30), ("cos", 2500, 33, 3, 1e-8), ("manh", 2500, 64, 2, 0.01), ("canb", 2001, 130, 3, 1e-12),
    ("eucl", 2003, 256, 3, 1e-30), ("cos", 2000, 200, 2, 1e-12), ("cos", 270_000, 66, 2, 1e-6),
    ("eucl", 300_001, 5, 2, 1e-16), ("manh", 530_000, 4, 3, 0.01)])
def test_split_w_pass(metric, n, d, k, delta):
    t, seed = 64, 3
    X, L = synth.tiny_case(n, d, k, seed=d)
    print(f"w pass metric={metric} d={d} n={n} k={k} delta={delta}", flush=True)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, metric, "fp32", t=t, delta=delta, seed=seed)
    native.silh_pps_sample(ctx)
    view = native.silh_sample_view(ctx)
    smp = oracle.sample(X, L, k, metric, t, delta, seed)
    assert_same_sets(smp, view, n, seed, "pps", t)
    for j in range(k):
        lo, hi = view["f0_offsets"][j], view["f0_offsets"][j + 1]
        assert hi > lo
        assert np.array_equal(view["f0_gid"][lo:hi], smp["F0"][j])
        np.testing.assert_allclose(view["f0_W"][lo:hi], smp["W0"][j], rtol=1e-13)
    np.testing.assert_allclose(view["p"], smp["p"], rtol=1e-13)
    native.silh_destroy(ctx)
