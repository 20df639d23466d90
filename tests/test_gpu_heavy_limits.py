"""GPU: the heavy phase of one launch at the limits of its rule (the bound of 640
heavy vertices, 448 vertices that may all be heavy), against the oracle, with its
launch asserted."""
import numpy as np
import pytest

import oracle
import synth
from synth import special
from test_gpu_plain_lists import _launches

pytestmark = pytest.mark.gpu


def _check(gpu, graph, split, small):
    n, src, dst = graph
    print("heavy limits", n, len(src), split, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g, heavy=split), "heavy_small", "heavy_mfma")
    want = oracle.count_split(og, *split)
    assert {k: got[k] for k in want} == want
    assert ran == [small, 1 - small]
    return got


# the bound is floor(2 m^1/2 + 2): 639, 640 and 641
@pytest.mark.parametrize("k,small", [(451, 1), (452, 1), (453, 0)])
def test_bound(gpu, k, small):
    _, src, dst = special.complete(k)
    ids = np.random.RandomState(k).permutation(2000)[:k].astype(np.int32)
    assert _check(gpu, (2000, ids[src], ids[dst]), (1, 1), small)["n_heavy"] == k


# bounds of 640 and 641 with few heavy vertices, and rows of every length
@pytest.mark.parametrize("m,split,small", [(101761, (1, 1), 1), (102081, (1, 1), 0), (25440, (1, 2), 1), (25521, (1, 2), 0)])
def test_sparse_bound(gpu, m, split, small):
    n = 20000
    _, a, b = synth.rmat(14, 5, seed=m)
    pairs = np.unique(np.sort(np.stack([a, b], 1)[a != b], 1), axis=0)
    _, c, d = synth.uniform_pairs(n, 150000, 1)
    more = np.unique(np.sort(np.stack([c, d], 1)[c != d], 1), axis=0)
    keep = more[~np.isin(more[:, 0] * np.int64(n) + more[:, 1], pairs[:, 0] * np.int64(n) + pairs[:, 1])]
    pairs = np.concatenate([pairs, np.random.RandomState(m).permutation(keep)])[:m]
    got = _check(gpu, (n, pairs[:, 0].astype(np.int32), pairs[:, 1].astype(np.int32)), split, small)
    assert got["m"] == m and got["n_heavy"] > 0


@pytest.mark.parametrize("n,small", [(2, 1), (33, 1), (256, 1), (448, 1), (449, 0), (640, 0)])
def test_all_may_be_heavy(gpu, n, small):
    for split in ((1, 1), (0, 1)):
        _check(gpu, special.complete(n), split, small)
