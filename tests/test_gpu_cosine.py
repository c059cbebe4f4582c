"""The cosine Phase 2 (cluster samples collapsed to one record each) against
the sum over pairs written out: operands rounded as the pairs' are (bf16, e4m3
times 64), pairs clamped to [0, 2] (fp8: the self pair), float64 sums; block and row-width
edges, a zero row, duplicate rows, a tight cluster and an empty one."""
import numpy as np
import pytest
import torch

from parity_util import dev
from paper_2607_01993_amd import native

pytestmark = pytest.mark.gpu


def _rows(n, d, k, seed):
    rng = np.random.default_rng(seed)
    mu = rng.standard_normal((k, d))
    L = rng.integers(0, k - 1, size=n).astype(np.int32)   # cluster k - 1 stays empty
    X = mu[L] + 0.6 * rng.standard_normal((n, d))
    tight = L == 0
    X[tight] = mu[0] + 1e-3 * rng.standard_normal((int(tight.sum()), d))
    X[1] = X[0]
    L[1] = L[0]
    X[5] = 0.0
    L[2], L[3], L[4] = 0, 1 % (k - 1), 0
    return np.ascontiguousarray(X.astype(np.float32)), L


def _pairs(X, L, k, prec):
    """W [n][k] by pairs, from the float32 unit rows the library forms."""
    # the reciprocal norm in float32 as the library states it (a fused chain in
    # coordinate order, rounded square root and division): an ulp of it would
    # move operands across rounding boundaries
    s2 = np.zeros(X.shape[0], dtype=np.float32)
    for c in range(X.shape[1]):
        s2 = (s2.astype(np.float64) + X[:, c].astype(np.float64) ** 2).astype(np.float32)
    one = np.float32(1.0)
    rn = torch.from_numpy(np.where(s2 > 0, one / np.sqrt(np.where(s2 > 0, s2, one)), np.float32(0.0)))
    X = torch.from_numpy(X)
    U = X * rn[:, None]
    u = torch.where(rn > 0, 0.0, 0.5).double()
    W = torch.zeros((X.shape[0], k), dtype=torch.float64)
    for j in range(k):
        ids = torch.nonzero(torch.from_numpy(L) == j)[:, 0]
        if ids.numel() == 0:
            continue
        c = U[ids].double()
        c = (c if prec == "fp32" else c[:256]).mean(dim=0).float()
        x, y = U - c, U[ids] - c
        if prec == "bf16":
            xq, yq = x.bfloat16().double(), y.bfloat16().double()
            nx, ny = (xq ** 2).sum(dim=1), (yq ** 2).sum(dim=1)
        elif prec == "fp8":
            xq = (64.0 * x).to(torch.float8_e4m3fn).double() / 64.0
            yq = (64.0 * y).to(torch.float8_e4m3fn).double() / 64.0
            nx, ny = (x.double() ** 2).sum(dim=1), (y.double() ** 2).sum(dim=1)
        else:
            xq, yq = x.double(), y.double()
            nx, ny = (xq ** 2).sum(dim=1), (yq ** 2).sum(dim=1)
        D = 0.5 * nx[:, None] + 0.5 * ny[None, :] + u[:, None] + u[None, ids] - xq @ yq.T
        # fp8: the sum is over the unclamped pairs and the clamped self pair
        self_pair = ids[None, :] == torch.arange(X.shape[0])[:, None]
        W[:, j] = torch.where(self_pair | (prec != "fp8"), D.clamp(0.0, 2.0), D).sum(dim=1)
    return W.numpy()


@pytest.mark.parametrize("prec,n,d,k", [("fp32", 63, 1, 3), ("fp32", 64, 8, 3), ("fp32", 129, 33, 4),
                                        ("fp32", 700, 129, 5), ("fp32_valu", 200, 256, 3), ("bf16", 63, 3, 3),
                                        ("bf16", 65, 16, 4), ("bf16", 128, 40, 18), ("bf16", 900, 100, 5),
                                        ("bf16", 130, 256, 3), ("fp8", 64, 64, 3), ("fp8", 600, 101, 4),
                                        ("fp8", 127, 256, 20)])
def test_sums_equal_the_pairs(prec, n, d, k):
    print(f"cosine {prec} n={n} d={d} k={k}", flush=True)
    X, L = _rows(n, d, k, seed=n + d)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "cos", prec, t=n, seed=1)   # every cluster whole, p = 1
    native.silh_pps_sample(ctx)
    W = native.silh_weighted_sums(ctx).cpu().numpy().astype(np.float64)
    native.silh_destroy(ctx)
    ref = _pairs(X, L, k, prec.split("_")[0])
    # float32 chains of at most 256 steps with unit-size terms against a sum of
    # |C_j| distances: 256 * 2^-24 of the sum, and of |C_j| times the norm terms
    # where those nearly cancel; fp8 on a tight cluster clamps single pairs
    # (|v|^2 - v_q.v'_q below 0), which the collapsed sum does only for the
    # self pairs: there the pairs' own size bounds the difference
    sizes = np.bincount(L, minlength=k).astype(np.float64)
    tol = 1.6e-5 * (ref + 1e-3 * sizes[None, :])
    if prec == "fp8":
        tol[:, 0] += 1e-5 * sizes[0]
    assert W.shape == ref.shape
    assert np.all(np.abs(W - ref) <= tol), np.max((np.abs(W - ref) - tol))
    assert np.all(W[:, k - 1] == 0.0)
