"""The autotuner keeps the shapes of split and unsplit, bounded and unbounded
launches apart: what one caller measured does not set another's."""
import time

import pytest
import torch

from paper_2607_01993_amd import native, synth
from parity_util import dev

pytestmark = pytest.mark.gpu


def _ms(f):
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    f()
    torch.cuda.synchronize()
    return time.perf_counter() - t0


def test_scores_are_timed_apart_from_sums():
    n, d, k = 600_000, 32, 16
    X, L = synth.tiny_case(n, d, k, seed=9)
    Xd, Ld = dev(X, L)
    ctx = native.silh_sample_init(Xd, Ld, k, "eucl", "fp32", t=512, seed=1)
    native.silh_pps_sample(ctx)
    try:
        for mode in (2, 3):          # every kernel loaded
            native.silh_set_tuning(mode)
            native.silh_weighted_sums(ctx)
            native.silh_scores(ctx)
        native.silh_set_tuning(1)    # forgets what was measured
        native.silh_weighted_sums(ctx)
        first = _ms(lambda: native.silh_scores(ctx))
        later = min(_ms(lambda: native.silh_scores(ctx)) for _ in range(6))
        print(f"scores: first {first * 1e3:.2f} ms, later {later * 1e3:.2f} ms", flush=True)
        # the first call times two shapes twice: four launches beside its own
        assert first > 2.0 * later
    finally:
        native.silh_set_tuning(1)
        native.silh_destroy(ctx)


def test_sweep_tunes_split_and_unsplit_clusterings_apart():
    """k = 3 runs unsplit and k = 5 split: each has a request of its own that
    its shape was timed on, though their samples fall in one size class."""
    n, d, ks, t = 5000, 16, [3, 5], 48
    X, _ = synth.tiny_case(n, d, 4, seed=2)
    Xd = torch.from_numpy(X).cuda()
    L = torch.stack([torch.from_numpy(synth.voronoi_labels(X, synth.voronoi_centers(n, k, (9, k)))) for k in ks])
    g = native.SweepGraph(Xd, L.cuda().contiguous(), ks, "eucl", "bf16", t=t, seed=5, chains=1)
    try:
        (s0, S0), (s1, S1) = g.choice(0), g.choice(1)
        assert S0 > 0 and S1 > 0 and S0 != S1
    finally:
        g.close()
