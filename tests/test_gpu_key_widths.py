"""GPU: the CSR build on both sides of window keys of 32 bits (twice the bits of
an id less the window's), with one partition pass and with two, against the
oracle's normalisation (byte-identical)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


# one pass: W = 7 and 8 window bits of 20-bit ids; two: 9 and 10 of 21, 11 and 12 of 22
@pytest.mark.parametrize("n,pairs", [((1 << 20) - 1, 30000), ((1 << 20) - 1, 200000), ((1 << 21) - 5, 500000),
                                     ((1 << 21) - 5, 1000000), ((1 << 22) - 1, 2000000), (1 << 22, 2400000)])
@pytest.mark.parametrize("leaves", [0, 9000])
def test_key_widths(gpu, n, pairs, leaves):
    """leaves: a hub whose window lies above the LDS limit, and is sorted by digits."""
    _, a, b = synth.uniform_pairs(n, pairs - 2 * leaves, 9)
    src = np.concatenate([a, np.full(leaves, n - 1, np.int32), a[:leaves]])
    dst = np.concatenate([b, a[:leaves], b[:leaves]])
    print("key widths", n, len(src), leaves, flush=True)
    rp, col, deg = gpu.tc_graph_read(gpu.tc_build_csr(n, src, dst))
    _, orp, ocol = oracle.normalise(n, src, dst)
    assert np.array_equal(rp, orp) and np.array_equal(col, ocol) and np.array_equal(deg, np.diff(orp))
