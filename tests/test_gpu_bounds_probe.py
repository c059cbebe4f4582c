"""From 65,536 elements on a probe decides whether the Euclidean bounds serve a
request: scores, row subsets and captured sweeps are the same on both sides of
its decision (clusters far apart, touching, and labels that have nothing to do
with the data)."""
import numpy as np
import pytest
import torch

from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def _data(kind, n, d, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    L = torch.randint(0, k, (n,), generator=g, device="cuda")
    spread = {"apart": 12.0, "near": 1.5, "random": 6.0}[kind]
    X = spread * torch.rand((k, d), generator=g, device="cuda")[L] + torch.randn((n, d), generator=g, device="cuda")
    if kind == "random":
        L = torch.randint(0, k, (n,), generator=g, device="cuda")
    return X.contiguous(), L.to(torch.int32).contiguous()


@pytest.mark.parametrize("kind", ["apart", "near", "random"])
@pytest.mark.parametrize("n,d,k,t,prec", [(65_536, 8, 16, 400, "bf16"), (70_001, 40, 5, 600, "fp32"),
                                          (200_003, 16, 33, 100, "bf16"), (66_000, 200, 6, 700, "bf16"),
                                          (65_535, 16, 9, 300, "fp32")])
def test_scores_are_those_of_the_sums(kind, n, d, k, t, prec):
    print(f"bounds probe {kind} n={n} d={d} k={k} {prec}", flush=True)
    X, L = _data(kind, n, d, k, seed=n % 89)
    ctx = native.silh_sample_init(X, L, k, "eucl", prec, t=t, seed=5)
    S, _ = native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    res = {x: v.cpu().numpy() if x != "mean" else v for x, v in native.silh_scores(ctx).items()}
    rows = torch.arange(n - 1, -1, -1, dtype=torch.int32, device="cuda")
    sub = {x: v.cpu().numpy() if x != "mean" else v for x, v in native.silh_scores_rows(ctx, rows).items()}
    native.silh_destroy(ctx)
    lab = L.cpu().numpy()
    sizes = np.bincount(lab, minlength=k).astype(np.float64)
    e = np.arange(n)
    a = W[e, lab] / np.maximum(sizes[lab] - 1, 1)
    B = W / sizes[None, :]
    B[e, lab] = np.inf
    b = B.min(axis=1)
    # both sides round the same float64 sums once to float32
    assert np.all(np.abs(res["a"] - a) <= 2.0 ** -22 * a)
    assert np.all(np.abs(res["b"] - b) <= 2.0 ** -22 * b)
    for x in "abs":
        assert np.array_equal(sub[x], res[x][::-1]), x


def test_sweep_equals_the_requests():
    n, d, ks, t = 80_000, 24, [9, 20], 300
    X, _ = _data("apart", n, d, 20, seed=3)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    L = torch.stack([_data("apart", n, d, 20, seed=3)[1] % ks[0],
                     torch.randint(0, ks[1], (n,), generator=g, device="cuda").to(torch.int32)]).contiguous()
    graph = native.SweepGraph(X, L, ks, "eucl", "bf16", t=t, seed=5, chains=2)
    want = []
    for i, k in enumerate(ks):
        ctx = native.silh_sample_init(X, L[i].contiguous(), k, "eucl", "bf16", t=t, delta=0.01, seed=5)
        native.silh_pps_sample(ctx)
        want.append(native.silh_scores(ctx, a=False, b=False, s=False)["mean"])
        native.silh_destroy(ctx)
    try:
        for _ in range(3):
            got = graph.run()
            assert got["reruns"] == 0 and list(got["means"]) == want
    finally:
        graph.close()
