"""Blocks whose waves share elements and split the clusters (n up to 2^18,
d <= 32) against the float64 oracle, at the edges of a block (32 or 64
elements) and of the four waves' shares of the clusters."""
import numpy as np
import pytest

import oracle
from parity_util import compare_scores, dev
from paper_2607_01993_amd import native, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,k,prec,mode", [(31, 3, 4, "fp32", 2), (65, 8, 5, "fp32", 3), (97, 16, 7, "bf16", 2),
                                             (128, 31, 4, "bf16", 3), (1500, 32, 9, "fp32", 2),
                                             (2111, 17, 13, "bf16", 3), (900, 5, 6, "fp32", 0)])
def test_split_blocks(n, d, k, prec, mode):
    print(f"split n={n} d={d} k={k} {prec} mode={mode}", flush=True)
    X, L = synth.tiny_case(n, d, k, seed=n)
    Xd, Ld = dev(X, L)
    native.silh_set_tuning(mode)
    try:
        res = native.silh_exact(Xd, Ld, k, "eucl", prec)
    finally:
        native.silh_set_tuning(1)
    ref = oracle.exact(X, L, k, "eucl")
    compare_scores(res, ref, prec=prec)
    assert abs(res["mean"] - np.asarray(res["s"].cpu().numpy(), dtype=np.float64).mean()) <= 2.0 ** -22


@pytest.mark.parametrize("n,d,k", [(700, 16, 3), (1301, 9, 5), (333, 3, 2)])
def test_clusters_of_several_blobs(n, d, k):
    """Cells of more blobs than clusters: most near pairs are recomputed."""
    X, _ = synth.tiny_case(n, d, 4 * k, seed=n)
    L = synth.voronoi_labels(X, synth.voronoi_centers(n, k, (n, k)))
    print(f"several blobs n={n} d={d} k={k}", flush=True)
    Xd, Ld = dev(X, L)
    res = native.silh_exact(Xd, Ld, k, "eucl", "fp32")
    compare_scores(res, oracle.exact(X, L, k, "eucl"))
