"""GPU: triple sampling where its paths part: samples partitioned by hash or
not, extension lists longer than one round of a block, and closing searches in
lists whose ids are far from evenly spread, against the oracle (exact)."""
import numpy as np
import pytest

import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu


def _check(gpu, n, src, dst, samples, hybrid, p=1.0):
    print("triples", n, len(src), samples, hybrid, p, flush=True)
    r = gpu.tc_triple_estimate(gpu.tc_build_csr(n, src, dst), p, samples, hybrid=hybrid, sample_seed=3, triple_seed=8)
    og = oracle.normalise(n, src, dst)
    if p < 1.0:
        og = oracle.sample(og, p, 3)
    size, wsum, closed = oracle.triple_sample(og, hybrid, samples, 8)
    assert (r["size"], r["weight_sum"], r["closed"], r["m"]) == (size, wsum, closed, len(og[2]) // 2)
    assert r["estimate"] == oracle.triple_estimate(size, wsum, samples, p)


@pytest.mark.parametrize("samples", [(1 << 21) - 1, 1 << 21, (1 << 21) + 8191])
@pytest.mark.parametrize("hybrid", [False, True])
def test_partition_threshold(gpu, samples, hybrid):
    n, src, dst = synth.rmat(18, 16, seed=2)
    _check(gpu, n, src, dst, samples, hybrid)


@pytest.mark.parametrize("leaves", [8191, 8192, 8193, 20000])
def test_long_extension_list(gpu, leaves):
    ids = np.arange(1, leaves + 1)
    src = np.concatenate([np.zeros(leaves, np.int64), ids[:-1], ids[: leaves // 2]]).astype(np.int32)
    dst = np.concatenate([ids, ids[1:], ids[leaves // 2: 2 * (leaves // 2)]]).astype(np.int32)
    _check(gpu, leaves + 1, src, dst, 30000, True)


@pytest.mark.parametrize("where", ["low", "high", "ends"])
@pytest.mark.parametrize("p", [1.0, 0.5])
def test_clustered_ids(gpu, where, p):
    n, (_, a, b) = 1 << 20, synth.uniform_pairs(400, 30000, 5)
    if where == "high":
        a, b = n - 1 - a, n - 1 - b
    elif where == "ends":  # half of every list at either end of the ids
        a, b = (np.where(x % 2, n - 1 - x, x) for x in (a, b))
    _check(gpu, n, a.astype(np.int32), b.astype(np.int32), 50000, True, p)
    _check(gpu, n, a.astype(np.int32), b.astype(np.int32), 50000, False, p)


@pytest.mark.parametrize("samples", [(1 << 18) - 1, 1 << 18, 1 << 20])
def test_extension_index_threshold(gpu, samples):
    n, src, dst = synth.rmat(18, 16, seed=2)
    _check(gpu, n, src, dst, samples, True)


@pytest.mark.parametrize("leaves,hubs", [(65536, 1), (70001, 2), (200000, 3)])
def test_extension_index_of_few_long_lists(gpu, leaves, hubs):
    ids = np.arange(hubs, hubs + leaves)
    src = np.concatenate([np.repeat(np.arange(hubs), leaves), ids[:-1:2], np.arange(hubs - 1)]).astype(np.int32)
    dst = np.concatenate([np.tile(ids, hubs), ids[1::2], np.arange(1, hubs)]).astype(np.int32)
    _check(gpu, hubs + leaves, src, dst, 1 << 18, True)


def test_more_samples_than_a_grid_holds_threads(gpu):
    # every wedge of K_n is closed, so the estimate is exact for any samples
    n, src, dst = special.complete(40)
    samples = (1 << 32) + 5
    print("triples", n, samples, flush=True)
    r = gpu.tc_triple_estimate(gpu.tc_build_csr(n, src, dst), 1.0, samples, hybrid=False)
    assert (r["closed"], r["weight_sum"]) == (samples, 20 * samples)
    assert r["estimate"] == 40 * 39 * 38 / 6
