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


@pytest.mark.parametrize("n,pairs,w4,w16", [(1000, 90000, 1, 0), (300, 90000, 1, 0), (700, 190000, 1, 0)])
def test_long_lists_of_one_class(gpu, n, pairs, w4, w16):
    """No degree above 512: the shorter classes' launches, whatever the edges."""
    _check(gpu, synth.uniform_pairs(n, pairs, 5), (2, 1), dict(work_w4=w4, work_w16=w16))


def test_long_lists_of_all_classes(gpu):
    """A degree above 512 in a small graph: one launch."""
    n, a, b = special.complete(420)
    _check(gpu, (900, np.concatenate([a, np.zeros(600, np.int32)]), np.concatenate([b, np.arange(300, 900, dtype=np.int32)])),
           (2, 1), dict(work_w4=0, work_w16=1))
