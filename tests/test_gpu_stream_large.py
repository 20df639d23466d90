"""GPU: the semi-streaming variant where its draws are partitioned: both kinds
of draws, wedges alone, pairs alone, few heavy vertices, against the oracle
(every count equal, the estimate bit for bit)."""
import pytest

import oracle
import synth
from synth import special

pytestmark = pytest.mark.gpu

GRAPHS = {"rmat18": lambda: synth.rmat(18, 16, seed=2), "uniform": lambda: synth.uniform_pairs(1 << 18, 9 << 18, 3),
          "complete": lambda: special.complete(2100)}
_built = {}


def _graph(gpu, name):
    if name not in _built:
        G = GRAPHS[name]()
        _built[name] = gpu.tc_build_csr(*G), oracle.normalise(*G)
    return _built[name]


@pytest.mark.parametrize("name,d,heavy,light", [("rmat18", 1.0, True, True), ("rmat18", 0.002, True, True),
                                                ("uniform", 1.0, False, True), ("complete", 4.0, True, False),
                                                ("complete", 0.01, True, True)])
@pytest.mark.parametrize("draws", [(1 << 21) - 1, 1 << 21, (1 << 21) + 8191])
def test_matches_oracle(gpu, name, d, heavy, light, draws):
    print("stream", name, d, draws, flush=True)
    g, og = _graph(gpu, name)
    got = gpu.tc_stream_estimate(g, d, draws, seed=6)
    assert (got["heavy"] > 0, got["light_size"] > 0) == (heavy, light)
    assert got == oracle.stream_estimate(og, d, draws, 6)[0]
