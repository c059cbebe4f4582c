"""Cosine requests of the server run their Phase 2 in pieces of about a
millisecond with a wait between them, so that short kernels of other requests
behind them in a hardware queue get their turn: the results are the direct
call's, and a small request ends before a large one that came first."""
import pytest
import torch

from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def _data(n, d, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    L = torch.randint(0, k, (n,), generator=g, device="cuda").to(torch.int32)
    X = torch.randn((k, d), generator=g, device="cuda")[L.long()] + torch.randn((n, d), generator=g, device="cuda")
    return X, L


@pytest.mark.parametrize("prec,d,k,m", [("bf16", 256, 128, 0), ("fp8", 100, 700, 0), ("fp32", 20, 900, 0),
                                        ("fp8", 100, 700, 150_000)])
def test_pieces_equal_the_direct_call(prec, d, k, m):
    n, t = 300_001, 4
    print(f"cosine pieces {prec} d={d} k={k} m={m}", flush=True)
    X, L = _data(n, d, k, seed=d)
    ctx = native.silh_sample_init(X, L, k, "cos", prec, t=t, delta=0.01, seed=2)
    native.silh_pps_sample(ctx)
    if m:
        rows = native.silh_draw_rows(2, n, m)
        mean = native.silh_scores_rows(ctx, rows, a=False, b=False, s=False)["mean"]
    else:
        mean = native.silh_scores(ctx, a=False, b=False, s=False)["mean"]
    native.silh_destroy(ctx)
    srv = native.Server(workers=1, hbm_budget_bytes=32 << 30)
    res = srv.wait(srv.submit(srv.add_dataset(X), L, k, "cos", prec, t=t, seed=2, m=m))
    srv.close()
    assert res["status"] == "SILH_OK" and res["s_mean"] == mean


def test_small_requests_are_not_held_behind_a_large_cosine_one():
    X, L = _data(4_000_000, 128, 1024, seed=1)
    Xs, Ls = _data(20_000, 16, 8, seed=2)
    srv = native.Server(workers=4, hbm_budget_bytes=64 << 30)
    ib, is_ = srv.add_dataset(X), srv.add_dataset(Xs)
    for _ in range(2):                     # the first time the workers' memory is warmed up
        tb = srv.submit(ib, L, 1024, "cos", "bf16", "uni", t=8, seed=1)
        ts = [srv.submit(is_, Ls, 8, "eucl", "bf16", t=64, seed=10 + i) for i in range(8)]
        rs, rb = [srv.wait(t) for t in ts], srv.wait(tb)
    srv.close()
    assert rb["status"] == "SILH_OK" and all(r["status"] == "SILH_OK" for r in rs)
    ms = [(r["done_ns"] - r["submit_ns"]) / 1e6 for r in rs + [rb]]
    print(f"large {ms[-1]:.1f} ms, small max {max(ms[:-1]):.1f} ms", flush=True)
    assert all(r["done_ns"] < rb["done_ns"] for r in rs)
