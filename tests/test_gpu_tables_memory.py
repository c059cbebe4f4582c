"""Manhattan and Canberra requests whose tables' buffers cannot be had take the
direct sums: they are served, within the float32 bounds of the oracle."""
import pytest

import oracle
from paper_2607_01993_amd import native, synth
from parity_util import compare_scores, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric,d", [("manh", 9), ("canb", 32), ("manh", 130)])
def test_no_memory_for_tables(metric, d, monkeypatch):
    n, k = 1500, 3
    X, L = synth.tiny_case(n, d, k, seed=d)
    print(f"tables refused metric={metric} d={d}", flush=True)
    Xd, Ld = dev(X, L)
    sizes, refused = [], []

    def alloc(nbytes, user):
        sizes.append(nbytes)
        if refuse is not None and len(sizes) == refuse:
            refused.append(nbytes)
            return None
        return native._py_alloc(nbytes, user)

    cb = native.ALLOC_FN(alloc)
    monkeypatch.setattr(native, "_ALLOC_CB", cb)
    refuse = None
    native.silh_exact(Xd, Ld, k, metric, "fp32")
    refuse = len(sizes)  # the request's last buffers are the tables'
    sizes.clear()
    got = native.silh_exact(Xd, Ld, k, metric, "fp32")
    assert refused
    compare_scores(got, oracle.exact(X, L, k, metric))
