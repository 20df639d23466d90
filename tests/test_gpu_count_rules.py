"""GPU: counts on both sides of the rules that choose hubs, the partition of the
v-major pairs and the launches of the long lists, against the oracle, with the
launches asserted."""
import numpy as np
import pytest

import light_schedule
import oracle
import synth
from synth import special
from test_gpu_plain_lists import _launches

pytestmark = pytest.mark.gpu

NAMES = ("hub_ids", "light_bits", "vmajor_place", "work_w4", "work_w16")


def _check(gpu, graph, split, expect, p=1.0):
    n, src, dst = graph
    print("count rules", n, len(src), split, p, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    if p < 1.0:
        got, ran = _launches(gpu, lambda: gpu.tc_estimate(g, p, [3], heavy=split)[0][0], *NAMES)
        og = oracle.sample(og, p, 3)
    else:
        got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g, heavy=split), *NAMES)
    want = oracle.count_split(og, *split)
    assert {k: got[k] for k in want} == want
    sched = light_schedule.light_work(og, *split, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])
    ran = dict(zip(NAMES, ran))
    assert {k: ran[k] for k in expect} == expect


def _uniform_and_hub(n, pairs, leaves, seed):
    _, a, b = synth.uniform_pairs(n, pairs, seed)
    hub = np.random.RandomState(seed).permutation(n)[:leaves + 1].astype(np.int32)
    return n, np.concatenate([a, np.full(leaves, hub[0], np.int32)]), np.concatenate([b, hub[1:]])


@pytest.mark.parametrize("hub,numbered", [(40, 0), (1200, 1)])
@pytest.mark.parametrize("p", [1.0, 0.9])
def test_skew(gpu, hub, numbered, p):
    """66000 vertices of degree 90 or so: hubs are numbered if one has four times the mean."""
    _check(gpu, _uniform_and_hub(66000, 3000000, hub, 1), (1, 1), dict(hub_ids=numbered, light_bits=numbered), p)


@pytest.mark.parametrize("pairs,hub,placed", [(870000, 1, 0), (870000, 1000, 1), (1600000, 1, 1)])
def test_sparse(gpu, pairs, hub, placed):
    """Past 786432 edges: below two a vertex the pairs are placed by partition only in a skewed graph."""
    _check(gpu, _uniform_and_hub(600000, pairs, hub, 2), (1, 1), dict(vmajor_place=placed))


@pytest.mark.parametrize("split", [(1, 1), (0, 1), (2, 1)])
def test_all_may_be_heavy(gpu, split):
    """K_1300, more edges than the partition's limit: no hubs and no partition where all vertices may be heavy."""
    on = 1 if split == (2, 1) else 0  # a bound of 920
    _check(gpu, special.complete(1300), split, dict(light_bits=on, vmajor_place=on))


@pytest.mark.parametrize("n,pairs,w4,w16", [(1000, 90000, 1, 0), (300, 90000, 1, 0), (700, 190000, 1, 0)])
def test_long_lists_of_one_class(gpu, n, pairs, w4, w16):
    """No degree above 512: the shorter classes' launches, whatever the edges."""
    _check(gpu, synth.uniform_pairs(n, pairs, 5), (2, 1), dict(work_w4=w4, work_w16=w16))


def test_long_lists_of_all_classes(gpu):
    """A degree above 512 in a small graph: one launch."""
    n, a, b = special.complete(420)
    _check(gpu, (900, np.concatenate([a, np.zeros(600, np.int32)]), np.concatenate([b, np.arange(300, 900, dtype=np.int32)])),
           (2, 1), dict(work_w4=0, work_w16=1))
