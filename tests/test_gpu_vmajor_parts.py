"""GPU: v-major pairs placed by partition at its limits: parts of 2^13 vertices,
which fill a record's bits, parts with many times the mean's records, and one
vertex past the largest graph it takes, against the oracle and the schedule model,
with the partition's launch asserted."""
import numpy as np
import pytest

import light_schedule
import oracle
from test_gpu_plain_lists import _launches

pytestmark = pytest.mark.gpu


def _skewed(n, power, pairs, core, core_pairs, seed):
    """Ids of density i^(1/power - 1), and a dense core of light vertices with long lists."""
    rng = np.random.RandomState(seed)
    e = (n * rng.rand(2, pairs) ** power).astype(np.int32)
    ids = rng.permutation(n)[:core]
    c = ids[rng.randint(core, size=(2, core_pairs))]
    return n, np.concatenate([e[0], c[0]]).astype(np.int32), np.concatenate([e[1], c[1]]).astype(np.int32)


@pytest.mark.parametrize("n,placed", [((1 << 22) - 3, 1), (1 << 22, 1), ((1 << 22) + 1, 0)])
@pytest.mark.parametrize("power", [1, 5])
def test_widest_parts(gpu, n, placed, power):
    n, src, dst = _skewed(n, power, 1500000, 1500, 400000, power)
    print("widest parts", n, power, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g), "vmajor_place", "light_large")
    want = oracle.count_split(og)
    assert {k: got[k] for k in want} == want and ran == [placed, 1] and got["items_large"] > 0
    sched = light_schedule.light_work(og, 1, 1, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])


@pytest.mark.parametrize("n,power,bits", [(30011, 3, 1), (200003, 6, 1), (600011, 8, 0)])
@pytest.mark.parametrize("p", [1.0, 0.8])
def test_few_parts_hold_most_pairs(gpu, n, power, bits, p):
    n, src, dst = _skewed(n, power, 2500000, 1200, 300000, n)
    print("uneven parts", n, power, p, flush=True)
    g, og = gpu.tc_build_csr(n, src, dst), oracle.normalise(n, src, dst)
    if p < 1.0:
        got, ran = _launches(gpu, lambda: gpu.tc_estimate(g, p, [5], heavy=(1, 2))[0][0], "vmajor_place", "light_bits")
        og = oracle.sample(og, p, 5)
    else:
        got, ran = _launches(gpu, lambda: gpu.tc_count_exact(g, heavy=(1, 2)), "vmajor_place", "light_bits")
    want = oracle.count_split(og, 1, 2)
    assert {k: got[k] for k in want} == want and ran == [1, bits]
    sched = light_schedule.light_work(og, 1, 2, 1024)
    assert (got["probes"], got["gather"]) == (sched["probes"], sched["gather"])
