"""GPU: the CSR build where a row's neighbours are bunched, around the number of
keys of a sub-window from which its window is sorted by digits, for windows of
one, two and four digits, against the oracle's normalisation."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(250, 40), (20000, 300), (1 << 19, 700)])
@pytest.mark.parametrize("bunch", [23, 24, 25, 47, 48, 49, 95, 96, 97, 130])
def test_bunches(gpu, n, rows, bunch):
    """Every row holds `bunch` consecutive ids and as many spread ones, each pair twice, in a shuffled order."""
    rng = np.random.RandomState(bunch)
    src = np.repeat(rng.choice(n, rows, replace=False), 2 * bunch).reshape(rows, 2, bunch)
    dst = np.stack([(rng.randint(n, size=(rows, 1)) + np.arange(bunch)) % n, rng.randint(n, size=(rows, bunch))], 1)
    order = rng.permutation(2 * src.size) % src.size
    src, dst = src.reshape(-1)[order].astype(np.int32), dst.reshape(-1)[order].astype(np.int32)
    print("csr bunched", n, rows, bunch, flush=True)
    rp, col, deg = gpu.tc_graph_read(gpu.tc_build_csr(n, src, dst))
    _, orp, ocol = oracle.normalise(n, src, dst)
    assert np.array_equal(rp, orp) and np.array_equal(col, ocol) and np.array_equal(deg, np.diff(orp))


@pytest.mark.parametrize("left", [100, 500, 1500, 2000])
def test_complete_bipartite(gpu, left):
    """Every list of the right side is the ids 0 .. left - 1."""
    right = 20000
    src, dst = np.repeat(np.arange(left, dtype=np.int32), right), np.tile(np.arange(left, left + right, dtype=np.int32), left)
    print("csr bipartite", left, right, flush=True)
    rp, col, deg = gpu.tc_graph_read(gpu.tc_build_csr(left + right, src, dst))
    assert np.array_equal(rp, np.concatenate([np.arange(left) * right, left * right + np.arange(right + 1) * left]))
    assert np.array_equal(col[:left * right], dst) and np.array_equal(col[left * right:], np.tile(np.arange(left, dtype=np.int32), right))
    assert np.array_equal(deg, np.diff(rp))
