"""GPU: the estimators' bucket index where one vertex's range holds whole groups
of buckets, with and without the index, against the oracle (exact)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _hubs(n, hubs, leaves, seed):
    """`hubs` vertices with many leaves each, among n - hubs of small degree."""
    rng = np.random.RandomState(seed)
    ids = rng.permutation(n)
    a, b = rng.randint(n, size=(2, n // 2))
    h = np.repeat(ids[:hubs], leaves)
    return n, np.concatenate([h, a]).astype(np.int32), np.concatenate([rng.randint(n, size=len(h)), b]).astype(np.int32)


# 2^15 - 1: an index without groups; 2^16: the first with them
@pytest.mark.parametrize("n,hubs,leaves", [((1 << 15) - 1, 1, 3000), (1 << 16, 1, 3000), (65537, 2, 2000),
                                           (200001, 1, 300), (200001, 40, 1000), (1 << 20, 1, 4000)])
def test_long_ranges(gpu, n, hubs, leaves):
    n, src, dst = _hubs(n, hubs, leaves, n + hubs)
    print("long ranges", n, hubs, leaves, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    for samples in (n // 8 - 1, n // 8, 300000):  # the index begins at an eighth of the vertices
        for hybrid in (False, True):
            r = gpu.tc_triple_estimate(g, 1.0, samples, hybrid=hybrid, triple_seed=5)
            assert (r["size"], r["weight_sum"], r["closed"]) == oracle.triple_sample(og, hybrid, samples, 5)
    assert gpu.tc_stream_estimate(g, 0.001, 200000, seed=3) == oracle.stream_estimate(og, 0.001, 200000, 3)[0]


@pytest.mark.parametrize("n", [1 << 16, (1 << 20) + 1])
def test_one_star(gpu, n):
    """All upper edges are vertex 0's: every bucket lies in a whole group."""
    src, dst = np.zeros(n - 1, np.int32), np.arange(1, n, dtype=np.int32)
    print("star", n, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    assert gpu.tc_stream_estimate(g, 1.0, 200000, seed=3) == oracle.stream_estimate(og, 1.0, 200000, 3)[0]
