"""GPU: small graphs, whose heavy phase is one block, around the sizes where
the one-block phase, the one-launch scans and the split windows begin and end:
counts and splits equal to the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu


def _check(gpu, n, src, dst, splits):
    print("small", n, len(src), splits, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    for a, b in splits:
        got, want = gpu.tc_count_exact(g, heavy=(a, b)), oracle.count_split(og, a, b)
        assert {k: got[k] for k in want} == want, (a, b)


@pytest.mark.parametrize("k", [3, 31, 32, 33, 64, 200, 451, 453, 460])
def test_cliques(gpu, k):
    """All vertices heavy; the bound of 640 heavy vertices lies at a clique of 452."""
    _check(gpu, *special.complete(k), splits=((1, 1), (1, 2), (2, 1), (0, 1)))


@pytest.mark.parametrize("n", [4095, 4097, 16383, 16384, 16385, 65535, 65536, 65537, 70000])
def test_vertex_counts(gpu, n):
    _, s, d = synth.rmat(10, 16, seed=n)
    e = np.random.RandomState(n).randint(n, size=(2, 60000)).astype(np.int32)
    _check(gpu, n, np.concatenate([s, e[0]]), np.concatenate([d, e[1]]), splits=((1, 1), (1, 4), (3, 1)))


@pytest.mark.parametrize("scale", [10, 12, 14])
def test_skewed(gpu, scale):
    _check(gpu, *synth.rmat(scale, 12, seed=7), splits=((1, 1), (1, 8), (1000, 1)))
