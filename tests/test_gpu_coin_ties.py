"""GPU: thresholds that agree with an edge's coin in the bits that decide
first, so that only the low bits tell whether the edge is kept."""
import numpy as np
import pytest

import oracle
from synth import special

pytestmark = pytest.mark.gpu


def _turn(u, v, seed):
    """Smallest t for which p = t / 2**53 keeps the edge."""
    lo, hi = 0, 1 << 53
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if oracle.keep(u, v, seed, mid / 2.0**53) else (mid, hi)
    return hi


@pytest.mark.parametrize("u,v,seed", [(0, 1, 1), (3, 70, 5), (11, 12, 77)])
@pytest.mark.parametrize("step", [-(1 << 22), -(1 << 21), -1, 0, 1, 1 << 21])
def test_last_bits_decide(gpu, u, v, seed, step):
    n, s, d = special.complete(90)
    g, og = gpu.tc_build_csr(n, s, d), oracle.normalise(n, s, d)
    p = (_turn(u, v, seed) + step) / 2.0**53
    assert oracle.keep(u, v, seed, p) == (step >= 0)
    _, _, col = oracle.sample(og, p, seed)
    assert np.array_equal(gpu.tc_sample(g, p, seed).read()[1], col)
    for seeds in ([seed, seed + 1, seed], list(range(seed - 1, seed + 65))):
        per, _, _ = gpu.tc_estimate(g, p, seeds)
        assert [c["triangles"] for c in per] == [oracle.count(oracle.sample(og, p, x)) for x in seeds]
