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
