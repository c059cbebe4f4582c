"""float32 Euclidean sums from three bf16 pieces (d from 9 to 64): the widths'
edges, rows far from the origin and rows of tiny scale, against the float64
oracle at float32's tolerance."""
import numpy as np
import pytest

import oracle
from paper_2607_01993_amd import native, synth
from parity_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale,shift", [(1.0, 0.0), (1.0, 300.0), (1e-17, 0.0), (1e15, 0.0)])
@pytest.mark.parametrize("d", [9, 16, 17, 32, 33, 64])
def test_float32_sums(d, scale, shift):
    n, k = 700, 5
    X, L = synth.tiny_case(n, d, k, seed=d)
    X = ((X + shift) * scale).astype(np.float32)
    print(f"pieces d={d} scale={scale} shift={shift}", flush=True)
    Xd, Ld = dev(X, L)
    got = native.silh_exact(Xd, Ld, k, "eucl", "fp32")
    ref = oracle.exact(X, L, k, "eucl")
    # a pair's squared distance is off by at most eps (|x~|^2 + |y~|^2) over
    # the 2^-5 below which it is summed directly: 2^-17 of the distance
    for key in ("a", "b"):
        np.testing.assert_allclose(got[key].cpu().numpy(), ref[key], rtol=2.0 ** -17)
