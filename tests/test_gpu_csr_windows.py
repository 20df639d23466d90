"""GPU: the CSR build at the sizes where its windows, passes and key widths
change, against the oracle's normalisation (byte-identical), with the exact
count of the built graph where the oracle is quick (the stored neighbour
classes orient it)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _check(gpu, n, src, dst, count=False):
    src, dst = np.asarray(src, np.int32), np.asarray(dst, np.int32)
    print("csr", n, len(src), flush=True)
    g = gpu.tc_build_csr(n, src, dst)
    _, orp, ocol = og = oracle.normalise(n, src, dst)
    rp, col, deg = gpu.tc_graph_read(g)
    assert np.array_equal(rp, orp) and np.array_equal(col, ocol) and np.array_equal(deg, np.diff(orp))
    assert g.info() == dict(n=n, m=len(ocol) // 2, max_deg=int(np.diff(orp).max(initial=0)))
    if count:
        assert gpu.tc_count_exact(g)["triangles"] == oracle.count(og)


@pytest.mark.parametrize("pairs", [1, 2, 63, 64, 65, 2047, 2048, 2049, 4095, 4097, 8193, 16385])
@pytest.mark.parametrize("n", [2, 3, 257, 5000])
def test_small(gpu, n, pairs):
    _check(gpu, n, *synth.uniform_pairs(n, pairs, pairs + n)[1:], count=True)


@pytest.mark.parametrize("pairs", [(1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1500007])
@pytest.mark.parametrize("n", [700, 65535, 65537, 1000003])
def test_one_and_two_passes(gpu, n, pairs):
    _check(gpu, n, *synth.uniform_pairs(n, pairs, 3)[1:])


@pytest.mark.parametrize("leaves", [8190, 16383, 16384, 16385, 20480, 40001])
@pytest.mark.parametrize("n", [50000, 1 << 20])
def test_hub_windows(gpu, n, leaves):
    """A star whose hub's window lies around the LDS limit, with a path and every pair twice."""
    hub, leaf = n // 2, np.setdiff1d(np.arange(leaves + 1), [n // 2])[:leaves]
    src = np.concatenate([np.full(leaves, hub), leaf[:-1], leaf, leaf[:5000]])
    dst = np.concatenate([leaf, leaf[1:], np.full(leaves, hub), leaf[:5000]])
    _check(gpu, n, src, dst, count=True)


@pytest.mark.parametrize("copies", [4096, 16384, 16385, 100000])
def test_one_edge_many_times(gpu, copies):
    _check(gpu, 1000, np.full(copies, 7), np.full(copies, 993))


@pytest.mark.parametrize("n", [(1 << 23) - 3, (1 << 24) + 5, (1 << 27) + 1])
def test_wide_ids(gpu, n):
    """Window keys of 32 and of 64 bits; the hub's window above the LDS limit."""
    _, a, b = synth.uniform_pairs(n, 600000, 9)
    hub = np.full(30000, n - 1)
    _check(gpu, n, np.concatenate([a, hub]), np.concatenate([b, a[:30000]]))


def test_skewed(gpu):
    _check(gpu, *synth.rmat(17, 16, seed=6), count=True)


def test_bad_ids_and_empty(gpu):
    for bad in (-1, 1000, 2 ** 31 - 1):
        with pytest.raises(gpu.TcError):
            gpu.tc_build_csr(1000, np.array([1, bad, 3], np.int32), np.array([2, 5, 4], np.int32))
    for n in (0, 1, 9):
        _check(gpu, n, [], [])
    _check(gpu, 4, [1, 2, 2], [1, 2, 2])
    with pytest.raises(gpu.TcError):
        gpu.tc_build_csr(0, np.array([0], np.int32), np.array([0], np.int32))
