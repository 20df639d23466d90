"""GPU: batched seeds whose union leaves out the vertices of degree 1: graphs
of mostly leaves, odd numbers of remaining entries, components that fill their
256-vertex windows, samples that lose every edge; all counts and statistics
equal to the single-seed call's."""
import numpy as np
import pytest

import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu


def _pendants(core, per):
    """A clique with `per` leaves at every vertex."""
    n, s, d = special.complete(core)
    leaf = np.arange(core, core * (per + 1), dtype=np.int32)
    return core * (per + 1), np.concatenate([s, np.repeat(np.arange(core), per)]).astype(np.int32), \
        np.concatenate([d, leaf]).astype(np.int32)


GRAPHS = {
    "pendants": _pendants(12, 9),
    "pendants_256": _pendants(16, 15),
    "path": (600, np.arange(599, dtype=np.int32), np.arange(1, 600, dtype=np.int32)),
    "triangles_512": special.disjoint_union(*[special.complete(4) for _ in range(128)]),
    "matching": (1000, np.arange(0, 1000, 2, dtype=np.int32), np.arange(1, 1000, 2, dtype=np.int32)),
    "sparse": synth.chung_lu(20000, 3.0, 2.3, seed=9),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("heavy", [(1, 1), (2, 1), (1, 2)])
@pytest.mark.parametrize("p", [0.999, 0.6, 0.01])
def test_equal_to_single_seeds(gpu, name, heavy, p):
    n, s, d = GRAPHS[name]
    print("leaves", name, heavy, p, flush=True)
    g, og = gpu.tc_build_csr(n, s, d), oracle.normalise(n, s, d)
    seeds = [3, 4, 5, 6, 7, 99, 100]
    per, _, _ = gpu.tc_estimate(g, p, seeds, heavy=heavy)
    assert per == [gpu.tc_estimate(g, p, [sd], heavy=heavy)[0][0] for sd in seeds]
    assert [c["triangles"] for c in per] == [oracle.count(oracle.sample(og, p, sd)) for sd in seeds]
