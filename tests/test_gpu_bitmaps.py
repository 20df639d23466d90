"""GPU: block anchors closed through hub bitmaps, at the edges of their rule
and layout, against the oracle: graphs whose vertices are all hubs and graphs
that number them, anchors on both sides of the hub limit, lists around the
lane groups' steps, lists too long to sort, and hub-free fallbacks."""
import numpy as np
import pytest

import light_schedule
import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu


def _check(gpu, graph, splits=((1, 1), (1, 4)), p=None):
    n, src, dst = graph
    print("bitmaps", n, len(src), splits, p, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    for a, b in splits:
        if p is None:
            got, want, work = gpu.tc_count_exact(g, heavy=(a, b)), oracle.count_split(og, a, b), og
        else:
            got = gpu.tc_estimate(g, p, [5], heavy=(a, b))[0][0]
            work = oracle.sample(og, p, 5)
            want = oracle.count_split(work, a, b)
        assert {k: got[k] for k in want} == want, (a, b)
        sched = light_schedule.light_work(work, a, b, 1024)
        assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])


def _dense_core(n, core, pairs, seed):
    """A dense random core (out-lists of hundreds) spread over n ids, and a sparse rest."""
    rng = np.random.RandomState(seed)
    ids = rng.permutation(n)[:core]
    a, b = ids[rng.randint(core, size=pairs)], ids[rng.randint(core, size=pairs)]
    c, d = rng.randint(n, size=4 * n), rng.randint(n, size=4 * n)
    return n, np.concatenate([a, c]).astype(np.int32), np.concatenate([b, d]).astype(np.int32)


@pytest.mark.parametrize("n", [2000, 65535, 65536, 70001])
@pytest.mark.parametrize("p", [None, 0.6])
def test_hub_limit(gpu, n, p):
    _check(gpu, _dense_core(n, 1500, 400000, n), p=p)


@pytest.mark.parametrize("core", [140, 190, 260, 420])
def test_list_lengths(gpu, core):
    """Cliques: lists of every length below the clique's, through one small dense graph and a numbered one."""
    _check(gpu, special.complete(core), splits=((1, 1), (1000, 1)))
    n, s, d = special.complete(core)
    rng = np.random.RandomState(core)
    ids = rng.permutation(80000)[:n]
    e = rng.randint(80000, size=(2, 700000))
    _check(gpu, (80000, np.concatenate([ids[s], e[0]]).astype(np.int32),
                 np.concatenate([ids[d], e[1]]).astype(np.int32)), splits=((1000, 1),))


def test_more_anchors_than_hubs(gpu):
    """Every vertex has a long list: most block anchors lie past the hub limit and keep the hash tables."""
    rng = np.random.RandomState(1)
    n, k = 70000, 170
    near = (np.arange(n)[:, None] + rng.randint(1, 400, size=(n, k))) % n
    _check(gpu, (n, np.repeat(np.arange(n), k).astype(np.int32), near.reshape(-1).astype(np.int32)),
           splits=((1000, 1),))


@pytest.mark.parametrize("split", [(1, 1), (1000, 1)])
def test_unsorted_lists(gpu, split):
    """Out-lists above 1024 entries, which stay in id order and stream whole."""
    _check(gpu, _dense_core(90000, 2100, 2200000, 3), splits=(split,))


@pytest.mark.parametrize("n", [(1 << 13) * 3 + 5, 1 << 16, 300001])
@pytest.mark.parametrize("p", [None, 0.9])
def test_placed_by_partition(gpu, n, p):
    """Enough edges for v-major pairs to be placed by partition: parts of several widths, hubs with many pairs."""
    rng = np.random.RandomState(n)
    e = (n * rng.rand(2, 2000000) ** 3).astype(np.int32)
    _check(gpu, (n, e[0], e[1]), splits=((1, 1), (1000, 1)), p=p)
