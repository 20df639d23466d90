"""GPU: the CSR build at the most pairs it takes, all of one window of rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ids", [(40000, 2), (1 << 17, 4)])
def test_most_pairs_in_one_window(gpu, n, ids):
    """2^31 - 2 keys in the window of rows 0 .. ids - 1: its last places lie within one step of a block of 2^31."""
    pairs = (1 << 30) - 1
    print("csr limit", n, pairs, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(ids)
    src = torch.randint(ids, (pairs,), dtype=torch.int32, device="cuda", generator=gen)
    dst = torch.randint(1, ids, (pairs,), dtype=torch.int32, device="cuda", generator=gen) if ids > 2 else 1
    dst = (src + dst) % ids  # never a loop
    g = gpu.tc_build_csr(n, src, dst)
    del src, dst
    rp, col, deg = gpu.tc_graph_read(g)
    assert g.info() == dict(n=n, m=ids * (ids - 1) // 2, max_deg=ids - 1)
    assert col.tolist() == [v for u in range(ids) for v in range(ids) if v != u]
    assert deg.tolist() == [ids - 1] * ids + [0] * (n - ids)
    del g
    torch.cuda.empty_cache()
