"""Requests at the limit of their device memory: buffers that only save work
(the bounds' masks and records) can be refused."""
import numpy as np
import pytest
import torch

from paper_2607_01993_amd import native, synth

pytestmark = pytest.mark.gpu


class Refusing:
    """The binding's allocator, refusing its call number `at` (from 0), blocks
    of `most` bytes and more, or what would take it past `limit` bytes in use."""

    def __init__(self, monkeypatch):
        self.at, self.calls, self.bytes, self.most, self.limit = None, 0, [], None, None
        self.live, self.used, self.peak = {}, 0, 0
        self.cbs = native.ALLOC_FN(self._alloc), native.FREE_FN(self._free)
        monkeypatch.setattr(native, "_ALLOC_CB", self.cbs[0])
        monkeypatch.setattr(native, "_FREE_CB", self.cbs[1])

    def _alloc(self, nbytes, user):
        self.calls += 1
        if (self.at is not None and self.calls - 1 == self.at) or (self.most is not None and nbytes >= self.most) \
                or (self.limit is not None and self.used + nbytes > self.limit):
            return None
        self.bytes.append(nbytes)
        p = native._py_alloc(nbytes, user)
        self.live[p] = nbytes
        self.used += nbytes
        self.peak = max(self.peak, self.used)
        return p

    def _free(self, p, user):
        self.used -= self.live.pop(p)
        native._py_free(p, user)

    def __call__(self, f, at=None):
        self.at, self.calls, self.bytes = at, 0, []
        try:
            return f()
        except native.SilhError as e:
            assert e.name == "SILH_E_NOMEM", e.name
            return None


def _plain(res):
    return {x: v.cpu().numpy() if isinstance(v, torch.Tensor) else v for x, v in res.items()}


def _same(a, b):
    return all(np.array_equal(a[x], b[x]) for x in a)


@pytest.mark.parametrize("d,prec,k", [(16, "bf16", 12), (5, "fp32", 12), (200, "bf16", 200), (16, "bf16", 200)])
def test_scores_without_the_bounds_buffers(d, prec, k, monkeypatch):
    n = 40_000
    print(f"scarce bounds d={d} {prec} k={k}", flush=True)
    X, L = synth.tiny_case(n, d, k, seed=d)
    Xd, Ld = torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda()
    rows = torch.arange(0, n, 2, dtype=torch.int32, device="cuda")

    def scores():
        ctx = native.silh_sample_init(Xd, Ld, k, "eucl", prec, t=600, seed=5)
        try:
            S, _ = native.silh_pps_sample(ctx)
            assert n * S >= 1 << 24       # the bounds are in use
            return {**_plain(native.silh_scores(ctx)),
                    **{"r" + x: v for x, v in _plain(native.silh_scores_rows(ctx, rows)).items()}}
        finally:
            native.silh_destroy(ctx)

    alloc = Refusing(monkeypatch)
    scores()
    ref = alloc(scores)
    served = [i for i in range(alloc.calls) if (got := alloc(scores, i)) is not None and _same(got, ref)]
    # the records and masks of the scores, the masks of the rows
    print("served without allocation", served, flush=True)
    assert len(served) == 2
    # the rows' buffers in place of the masks, and of the scores' where those
    # have an allocation of their own
    alloc.peak = 0
    alloc(scores)
    for less in (1, (64 + -(-(n // 2) // 32) * -(-k // 32)) * 4 + 4096)[:2 if k > 128 else 1]:
        alloc.limit = alloc.peak - less
        got = alloc(scores)
        alloc.limit = None
        assert got is not None and _same(got, ref), less


def _hooked(monkeypatch):
    """SweepGraph through the allocator hooks (it takes its memory itself)."""
    plain = native._params
    monkeypatch.setattr(native, "_params", lambda *a, use_torch_alloc=True, **kw: plain(*a, use_torch_alloc=True, **kw))
    monkeypatch.setattr(native._alloc_state, "target", (0, torch.cuda.current_stream()), raising=False)


def test_sweep_without_the_bounds_buffers(monkeypatch):
    n, d, ks = 30_000, 16, [3, 9, 17]
    X = synth.exp_blobs(n, d, 5, seed=3)
    L = np.stack([synth.voronoi_labels(X, synth.voronoi_centers(n, k, (3, k))) for k in ks])
    Xd, Ld = torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda().contiguous()

    def sweep():
        g = native.SweepGraph(Xd, Ld, ks, "eucl", "bf16", t=400, seed=5, chains=1)
        try:
            return {"means": g.run()["means"]}
        finally:
            g.close()

    _hooked(monkeypatch)
    alloc = Refusing(monkeypatch)
    sweep()
    ref = alloc(sweep)
    # a record of 8 + 16 floats a cluster and 32 words, a mask word per 32 elements past a head of 64
    at = [i for i, b in enumerate(alloc.bytes) if b in ((17 * 24 + 32) * 4, (64 + -(-n // 32)) * 4)]
    assert len(at) >= 2
    for i in at:
        got = alloc(sweep, i)
        assert got is not None and _same(got, ref), i


@pytest.mark.parametrize("d", [12, 40])
def test_float32_without_the_larger_operand_rows(d, monkeypatch):
    """float32 Euclidean at d = 9 to 64 takes larger operand rows than float32
    itself: without memory for them the request, and a captured sweep, are
    served by the direct float32 sums."""
    n, k = 3000, 5
    print(f"scarce operands d={d}", flush=True)
    X, L = synth.tiny_case(n, d, k, seed=d)
    Xd, Ld = torch.from_numpy(X).cuda(), torch.from_numpy(L).cuda()

    def scores(prec="fp32"):
        return _plain(native.silh_exact(Xd, Ld, k, "eucl", prec))

    alloc = Refusing(monkeypatch)
    scores()
    ref = alloc(scores)
    direct = scores("fp32_valu")
    # rows of three bf16 pieces and the norms (past d = 32 a tail): more than
    # the rest of the sample's buffers together
    row = {12: 2 * (3 * 16 + 8), 40: 2 * (3 * 64 + 16) + 16}[d]
    assert max(alloc.bytes) >= row * n
    alloc.most = row * n
    got = alloc(scores)
    alloc.most = None
    assert got is not None and _same(got, direct)
    assert abs(got["mean"] - ref["mean"]) <= 2.0 ** -20      # float32 sums both

    _hooked(monkeypatch)
    Lk = Ld[None].contiguous()

    def sweep(prec="fp32"):
        g = native.SweepGraph(Xd, Lk, [k], "eucl", prec, t=64, seed=5, chains=1)
        try:
            return {"means": g.run()["means"]}
        finally:
            g.close()

    sweep()
    alloc(sweep)
    # the sweep's capacity: 4 k t rows and a block of padding per cluster
    at = alloc.bytes.index((4 * k * 64 + 32 * k) * row)
    want = sweep("fp32_valu")
    got = alloc(sweep, at)
    assert got is not None and _same(got, want)
