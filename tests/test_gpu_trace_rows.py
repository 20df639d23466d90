"""GPU: the trace's row products where the kernel branches: graphs with and
without stored neighbour classes, lists around the sizes of the 64-entry
batches, and row tables below and past 4 GiB, against the oracle (exact)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _star_pairs(n, centre, leaves):
    """A star with a triangle on every second leaf."""
    a = np.concatenate([np.full(len(leaves), centre), leaves[0:-1:2]])
    b = np.concatenate([leaves, leaves[1::2]])
    return a.astype(np.int32), b.astype(np.int32)


@pytest.mark.parametrize("leaves", [2, 62, 64, 66, 128, 4094, 4100])
def test_batches(gpu, leaves):
    n = leaves + 3
    src, dst = _star_pairs(n, 1, np.arange(3, n))
    print("trace batches", leaves, flush=True)
    q, est = gpu.tc_rp_trace(gpu.tc_build_csr(n, src, dst), 70, 5)
    oq, oest = oracle.rp_trace(oracle.normalise(n, src, dst), 70, 5)
    assert np.array_equal(q, oq) and est == oest


@pytest.mark.parametrize("p", [0.7, 0.05])
def test_sampled_graph(gpu, p):
    n, src, dst = synth.rmat(13, 16, seed=3)
    print("trace of a sampled graph", p, flush=True)
    g = gpu.tc_sample(gpu.tc_build_csr(n, src, dst), p, 4)
    q, est = gpu.tc_rp_trace(g, 65, 9)
    oq, oest = oracle.rp_trace(oracle.sample(oracle.normalise(n, src, dst), p, 4), 65, 9)
    assert np.array_equal(q, oq) and est == oest


@pytest.mark.parametrize("n", [(1 << 24) - 1, (1 << 24) + 77])
@pytest.mark.parametrize("sampled", [False, True])
def test_row_table_around_4_gib(gpu, n, sampled):
    s, r, c = synth.uniform_pairs(3000, 20000, 7)
    src, dst = (np.concatenate([x, n - 1 - x]).astype(np.int32) for x in (r, c))
    print("trace rows", n, sampled, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    if sampled:
        g, og = gpu.tc_sample(g, 0.5, 2), oracle.sample(og, 0.5, 2)
    q, est = gpu.tc_rp_trace(g, 3, 1)
    oq, oest = oracle.rp_trace(og, 3, 1)
    assert np.array_equal(q, oq) and est == oest
