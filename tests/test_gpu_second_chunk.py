"""GPU: partitioned draws past one chunk of 2^26: what the draws of the second
chunk add, against the oracle's elements one by one (exact)."""
import numpy as np
import pytest

import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu

CHUNK, MORE, SEED = 1 << 26, 3001, 11


@pytest.mark.parametrize("hybrid", [False, True])
def test_triples(gpu, hybrid):
    G = synth.rmat(18, 16, seed=2)
    g, og = gpu.tc_build_csr(*G), oracle.normalise(*G)
    print("second chunk, triples", hybrid, flush=True)
    one, two = (gpu.tc_triple_estimate(g, 1.0, s, hybrid=hybrid, triple_seed=SEED) for s in (CHUNK, CHUNK + MORE))
    size, pre = oracle.triples_size(og, hybrid, with_prefix=True)
    w = [oracle.triple_at(og, hybrid, pre, oracle.triple_index(SEED, CHUNK + i, size))[1] for i in range(MORE)]
    assert one["size"] == two["size"] == size
    assert two["weight_sum"] - one["weight_sum"] == sum(w)
    assert two["closed"] - one["closed"] == sum(x > 0 for x in w) > 0


@pytest.mark.parametrize("d", [0.01, 1.0])
def test_stream(gpu, d):
    """On a complete graph every wedge is closed, and a pair unless its vertex is in its edge."""
    G = special.complete(2100)
    g, og = gpu.tc_build_csr(*G), oracle.normalise(*G)
    print("second chunk, stream", d, flush=True)
    one, two = (gpu.tc_stream_estimate(g, d, s, seed=SEED) for s in (CHUNK, CHUNK + MORE))
    want, heavy = oracle.stream_estimate(og, d, 0, SEED)
    hl, (v, w) = np.flatnonzero(heavy), np.triu_indices(2100, 1)
    closed = queries = 0
    salt = oracle.mix64(SEED ^ 0x54435F5354524D32)
    for i in range(CHUNK, CHUNK + MORE):
        r = (oracle.mix64(oracle.mix64(i) ^ salt) * want["size"]) >> 64
        if r < want["light_size"]:
            closed, queries = closed + 1, queries + 1
        else:
            h, e = divmod(r - want["light_size"], want["m"])
            if hl[h] not in (v[e], w[e]):
                closed, queries = closed + 1, queries + 2
    assert (two["size"], two["light_size"]) == (want["size"], want["light_size"])
    assert (two["closed"] - one["closed"], two["queries"] - one["queries"]) == (closed, queries)
