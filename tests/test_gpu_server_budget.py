"""Requests that fit the server's memory budget only without what saves work:
they are served without it, inside the budget."""
import threading

import pytest
import torch

from paper_2607_01993_amd import native, synth

pytestmark = pytest.mark.gpu


def _mean(Xd, Ld, k, metric, prec, t):
    ctx = native.silh_sample_init(Xd, Ld, k, metric, prec, t=t, delta=0.01, seed=3)
    try:
        native.silh_pps_sample(ctx)
        return native.silh_scores(ctx, a=False, b=False, s=False)["mean"]
    finally:
        native.silh_destroy(ctx)


def _served(Xd, Ld, k, metric, prec, t, budget, batched):
    """The served mean and the device memory taken meanwhile, as seen by polling."""
    torch.cuda.synchronize()
    srv = native.Server(workers=2, hbm_budget_bytes=budget, batched=batched)
    did = srv.add_dataset(Xd)
    free0, low, stop = torch.cuda.mem_get_info()[0], [], threading.Event()

    def poll():
        while not stop.is_set():
            low.append(torch.cuda.mem_get_info()[0])

    th = threading.Thread(target=poll)
    th.start()
    try:
        res = srv.wait(srv.submit(did, Ld, k, metric, prec, t=t, seed=3))
    finally:
        stop.set()
        th.join()
        srv.close()
    assert res["status"] == "SILH_OK", res
    return res["s_mean"], free0 - min(low)


@pytest.mark.parametrize("batched", [True, False])
def test_manhattan_without_tables(batched, monkeypatch):
    n, d, k, t = 200_000, 64, 8, 512
    print(f"lean manh batched={batched}", flush=True)
    X, L = synth.tiny_case(n, d, k, seed=5)
    Xd, Ld = torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda()
    tables = _mean(Xd, Ld, k, "manh", "fp32", t)
    calls, refuse = [], []

    def alloc(nbytes, user):
        calls.append(nbytes)
        return None if refuse and len(calls) == refuse[0] else native._py_alloc(nbytes, user)

    cb = native.ALLOC_FN(alloc)
    monkeypatch.setattr(native, "_ALLOC_CB", cb)
    _mean(Xd, Ld, k, "manh", "fp32", t)
    refuse.append(len(calls))            # the request's last buffers are the tables'
    calls.clear()
    direct = _mean(Xd, Ld, k, "manh", "fp32", t)
    # about 54 MB without the tables, 120 MB more with them
    budget = 100_000_000
    mean, used = _served(Xd, Ld, k, "manh", "fp32", t, budget, batched)
    print(f"used {used / 1e6:.0f} MB of {budget / 1e6:.0f}", flush=True)
    assert mean == direct
    assert used <= budget
    mean, _ = _served(Xd, Ld, k, "manh", "fp32", t, 1 << 30, batched)
    assert mean == tables


@pytest.mark.parametrize("batched", [True, False])
def test_float32_without_the_larger_rows(batched):
    n, d, k, t = 20_000, 40, 64, 300
    print(f"lean eucl batched={batched}", flush=True)
    X, L = synth.tiny_case(n, d, k, seed=6)
    Xd, Ld = torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda()
    # 19.4 MB with float32 rows, 22.6 with rows of three pieces
    mean, _ = _served(Xd, Ld, k, "eucl", "fp32", t, 21_000_000, batched)
    assert mean == _mean(Xd, Ld, k, "eucl", "fp32_valu", t)
    mean, _ = _served(Xd, Ld, k, "eucl", "fp32", t, 1 << 30, batched)
    assert mean == _mean(Xd, Ld, k, "eucl", "fp32", t)
