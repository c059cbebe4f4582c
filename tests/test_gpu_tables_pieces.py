"""Manhattan and Canberra tables where they do not all fit at once: several
groups of tables (a cluster's parts on both sides of a group's end), elements
in several pieces, an empty cluster; and the pieces of a served request."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_01993_amd import native, synth
from test_gpu_tables_range import sums_and_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["manh", "canb"])
@pytest.mark.parametrize("n,t", [(60_000, 60_000), (140_000, 10_000)])
def test_groups_and_pieces(metric, n, t):
    """d = 256: a group is 27 tables of 1,024 rows (Manhattan 38), a piece
    131,072 elements; whole clusters of 20,000 rows are 20 tables each."""
    d, k = 256, 4
    print(f"tables groups {metric} n={n} t={t}", flush=True)
    rng = np.random.default_rng(n)
    L = rng.integers(0, 3, size=n).astype(np.int32)
    L[L == 2] = 3                          # cluster 2 stays empty
    X = (rng.uniform(0.5, 3.0, size=(k, d))[L] + rng.exponential(1.0, size=(n, d))).astype(np.float32)
    W, res, rows, ref = sums_and_pairs(X, L, k, metric, t, count=12)
    assert np.all(W[:, 2] == 0.0)
    on = [0, 1, 3]
    # a table's value to 2^-22 of itself, one rounding of the result
    assert np.all(np.abs(W[rows] - ref)[:, on] <= 2.0 ** -20 * ref[:, on])
    # elements on both sides of a piece's end: the scores are those of the sums
    a, b, s = oracle.silhouette.scores_from_weights(W, L, np.bincount(L, minlength=k))
    for x, v in zip("abs", (a, b, s)):
        assert np.max(np.abs(res[x].cpu().numpy() - v) - 2.0 ** -21 * np.abs(v)) <= (2.0 ** -20 if x == "s" else 0.0), x
    assert abs(res["mean"] - s.mean()) <= 2.0 ** -20


@pytest.mark.parametrize("metric,batched", [("manh", True), ("canb", True), ("canb", False)])
def test_served_pieces_equal_the_direct_call(metric, batched):
    n, d, k, t = 600_000, 64, 32, 60       # pieces of 262,144 elements
    print(f"tables served pieces {metric}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    Ld = torch.randint(0, k, (n,), generator=g, device="cuda").to(torch.int32)
    Xd = 0.5 + torch.rand((k, d), generator=g, device="cuda")[Ld.long()] \
        + torch.rand((n, d), generator=g, device="cuda")
    ctx = native.silh_sample_init(Xd, Ld, k, metric, "fp32", t=t, delta=0.01, seed=2)
    native.silh_pps_sample(ctx)
    mean = native.silh_scores(ctx, a=False, b=False, s=False)["mean"]
    native.silh_destroy(ctx)
    srv = native.Server(workers=1, hbm_budget_bytes=32 << 30, batched=batched)
    res = srv.wait(srv.submit(srv.add_dataset(Xd), Ld, k, metric, "fp32", t=t, seed=2))
    srv.close()
    assert res["status"] == "SILH_OK" and res["s_mean"] == mean
