"""Selections whose block counts feed the scan, with offsets and padded sizes
taken on the device, at the edges of 256-element blocks, 2048-element tiles and
of the largest count of tiles summed by the scan itself."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_01993_amd import native
from parity_util import assert_same_sets, dev

pytestmark = pytest.mark.gpu


def _case(n, k):
    rng = np.random.default_rng(n + k)
    L = np.minimum(np.arange(n), k - 1).astype(np.int32) if n < 2 * k else rng.integers(0, k, n).astype(np.int32)
    return rng.normal(size=(n, 3)).astype(np.float32), L


@pytest.mark.parametrize("sampler", ["pps", "uni"])
@pytest.mark.parametrize("n,k", [(2, 2), (255, 2), (256, 3), (257, 2), (2047, 5), (2048, 4), (2049, 1100), (4097, 70)])
def test_samples_at_edge_sizes(n, k, sampler):
    t, seed = 8, 5
    X, L = _case(n, k)
    print(f"scan edges n={n} k={k} sampler={sampler}", flush=True)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "eucl", "fp32", sampler, t=t, delta=0.1, seed=seed)
    native.silh_pps_sample(ctx)
    view = native.silh_sample_view(ctx)
    smp = oracle.sample(X, L, k, "eucl", t, 0.1, seed, sampler)
    assert_same_sets(smp, view, n, seed, sampler, t)
    np.testing.assert_allclose(view["p"], smp["p"], rtol=1e-13)
    native.silh_destroy(ctx)


@pytest.mark.parametrize("n", [2048 * 2048 - 1, 2048 * 2048 + 1])
def test_uniform_sample_of_many_tiles(n):
    k, t, seed = 3, 4000, 9
    X, L = _case(n, k)
    print(f"scan of many tiles n={n}", flush=True)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "eucl", "fp32", "uni", t=t, seed=seed)
    native.silh_pps_sample(ctx)
    view = native.silh_sample_view(ctx)
    native.silh_destroy(ctx)
    u = native.silh_philox_uniform(seed, 0, n, 2).cpu().numpy()
    sel = u < t / np.bincount(L)[L].astype(np.float64)
    want = [np.flatnonzero(sel & (L == j)) for j in range(k)]
    assert np.array_equal(view["gid"], np.concatenate(want))
    assert np.array_equal(np.diff(view["offsets"]), [len(w) for w in want])
