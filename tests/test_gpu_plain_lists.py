"""GPU: heavy vertices' lists of every length up to a clique's, in windows full
of them, streamed by light block anchors: against the oracle, with the kernels
that must have taken them asserted."""
import numpy as np
import pytest

import light_schedule
import oracle

pytestmark = pytest.mark.gpu


def _launches(gpu, call, *names):
    """call() and the launches of each of names during it."""
    gpu.profile.select(list(names))
    gpu.profile.reset()
    gpu.profile.enable(True)
    try:
        out = call()
    finally:
        gpu.profile.enable(False)
    got = [gpu.profile.read(k)[1] for k in names]
    gpu.profile.select(None)
    return out, got


def _core(core, light, each, n, seed):
    """A clique of the ids 0 .. core - 1 and `light` vertices joined to `each` of it, n vertices in all."""
    rng = np.random.RandomState(seed)
    i, j = np.triu_indices(core, 1)
    nb = np.argsort(rng.rand(light, core), 1)[:, :each]
    return n, np.concatenate([i, np.repeat(np.arange(core, core + light), each)]).astype(np.int32), \
        np.concatenate([j, nb.reshape(-1)]).astype(np.int32)


@pytest.mark.parametrize("core,light,n,split,placed", [(140, 700, 3000, (1, 1), 0), (700, 2000, 20000, (1, 1), 0),
                                                       (700, 2000, 70001, (1, 1), 0),
                                                       (1100, 3000, 20000, (1, 2), 1), (1100, 3000, 90000, (1, 2), 1)])
def test_core(gpu, core, light, n, split, placed):
    n, src, dst = _core(core, light, 130, n, core + n)
    print("plain lists", core, n, split, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g, heavy=split), "light_bits", "vmajor_place")
    want = oracle.count_split(og, *split)
    assert {k: got[k] for k in want} == want
    sched = light_schedule.light_work(og, *split, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])
    assert got["n_heavy"] == core and got["items_large"] > 0
    assert ran == [1, placed]


@pytest.mark.parametrize("n", [20000, 131072])
def test_long_streams(gpu, n):
    """Light lists of 700 entries stream parts of every length up to theirs, to bitmaps of names and of own ids."""
    n, src, dst = _core(1100, 1500, 700, n, n)
    ids = np.random.RandomState(n).permutation(n).astype(np.int32)
    print("long streams", n, flush=True)
    g, og = gpu.tc_build_csr(n, ids[src], ids[dst]), oracle.normalise(n, ids[src], ids[dst])
    got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g), "light_bits", "hub_ids")
    want = oracle.count_split(og)
    assert {k: got[k] for k in want} == want and ran == [1, n > 65535]
    sched = light_schedule.light_work(og, 1, 1, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])
    assert got["n_heavy"] == 1100 and got["items_large"] >= 1500


def _degree_class(d):
    """Degrees above 15 in eight steps an octave."""
    e = np.floor(np.log2(d)).astype(np.int64)
    return 8 * e + (d >> (e - 3) & 7)


def test_anchors_past_the_hubs(gpu):
    """Block anchors among the 65535 vertices of the highest classes and below them: bitmaps and tables in one count."""
    rng = np.random.RandomState(3)
    n, more = 80000, 20000
    near = (np.arange(n)[:, None] + rng.randint(1, 1500, size=(n, 150))) % n
    far = rng.permutation(n)[:more]
    pairs = far[rng.randint(more, size=(2, 60 * more))]
    hub = rng.permutation(n)[:2000]
    src = np.concatenate([np.repeat(np.arange(n), 150), pairs[0], np.full(2000, 5)]).astype(np.int32)
    dst = np.concatenate([near.reshape(-1), pairs[1], hub]).astype(np.int32)
    print("anchors past the hubs", len(src), flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g), "light_bits", "light_large", "hub_ids")
    want = oracle.count_split(og)
    assert {k: got[k] for k in want} == want and ran == [1, 1, 1]
    sched = light_schedule.light_work(og, 1, 1, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])
    # block anchors (more than 128 out-neighbours) of classes with numbers and without
    deg = np.diff(og[1])
    row, col = np.repeat(np.arange(n), deg), og[2]
    out = np.bincount(row[deg[row] * n + row < deg[col].astype(np.int64) * n + col], minlength=n)
    above = np.cumsum(np.bincount(_degree_class(deg))[::-1])[::-1]  # vertices of a class and above
    hubs = above[_degree_class(deg)] <= 65535
    anchors = (out > 128) & (deg.astype(np.int64) ** 2 <= got["m"])
    assert (anchors & hubs).sum() > 100 and (anchors & ~hubs).sum() > 100
