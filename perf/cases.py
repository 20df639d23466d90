"""The work that a program using this package has it do, as cases to be timed.

Every case is one call (or one burst of calls) of a public entry point on a
synthetic power-law graph.  The graphs are R-MAT (the shape of the paper's
social and web graphs, edge factor 16) and Chung-Lu (power-law expected
degrees), drawn on the device from the seed; vertex counts reach from a few
thousand (one request of a serving mix, where launches and synchronisations
count) to 2**22 (the benchmark's R-MAT scale 22).
"""
import math

import numpy as np
import torch

import paper_1011_0468_amd as tc

DEV = "cuda"
SERVE_P = (1.0, 0.5, 0.1)


def _case(name, kind, graph, n, pairs, **more):
    c = dict(name=name, kind=kind, graph=graph, n=n, pairs=pairs)
    c.update(more)
    return c


def listed():
    big = dict(n=1 << 22, pairs=1 << 26)
    return [
        # a new graph arrives: a small one, as one request of a service; and the benchmark's largest
        _case("build-10k", "build", "rmat", 10007, 160000),
        _case("build-rmat22", "build", "rmat", **big),
        # the exact count: latency of one small graph, an ordinary one of odd size, the largest with the
        # paper's own split
        _case("count-cl16k", "count", "chung-lu", 16384, 98304, p=1.0, heavy_num=1, heavy_den=1),
        _case("count-300k", "count", "rmat", 300007, 4800112, p=1.0, heavy_num=1, heavy_den=1),
        _case("count-rmat22", "count", "rmat", p=1.0, heavy_num=1, heavy_den=1, **big),
        # sparsify, then count: a dense sample with the split that the autotuner takes for it, and the
        # paper's headline p = 0.1
        _case("estimate-rmat22-half", "count", "rmat", p=0.5, heavy_num=1, heavy_den=4, **big),
        _case("estimate-rmat22-tenth", "count", "rmat", p=0.1, heavy_num=1, heavy_den=1, **big),
        # median of means over many seeds in one call
        _case("batch-cl20", "batch", "chung-lu", 1 << 20, 16 << 20, p=0.05, seeds=64, groups=8),
        # the random-projection trace of section 5.1
        _case("trace-rmat22", "trace", "rmat", k=128, **big),
        # triple sampling (the Hybrid column of Table 2) and the semi-streaming estimate of section 5.2
        _case("triples-rmat22", "triples", "rmat", p=1.0, samples=1 << 25, hybrid=True, **big),
        _case("stream-rmat22", "stream", "rmat", d=1.0, samples=1 << 24, **big),
        # a burst of independent requests (graph on the host, p and seed of its own) through the server
        _case("serve-48", "serve", "rmat", 1 << 18, 16 << 18, requests=48, lanes=4, fuse_max_pairs=262144),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "count", "count", "estimate", "estimate", "noalloc", "batch", "trace", "triples",
                       "stream", "serve"])
    graph = rng.choice(["rmat", "rmat", "chung-lu"])
    hi = {"batch": 1 << 18, "noalloc": 12000}.get(kind, 1 << 22)
    n = _log_uniform(rng, 3000, hi)
    pairs = n * (rng.randint(4, 8) if kind == "noalloc" else rng.randint(6, 16)) + rng.randint(0, 99)
    c = dict(kind=kind, graph=graph, n=n, pairs=pairs)
    heavy = rng.choice([(1, 1), (1, 1), (1, 2), (1, 4)])
    if kind in ("count", "estimate", "noalloc"):
        c.update(kind="noalloc" if kind == "noalloc" else "count",
                 p=1.0 if kind == "count" else round(math.exp(rng.uniform(math.log(0.05), math.log(0.9))), 4),
                 heavy_num=heavy[0], heavy_den=heavy[1])
    elif kind == "batch":
        groups = rng.choice([1, 4, 8])
        c.update(p=round(rng.uniform(0.05, 0.3), 4), seeds=groups * rng.randint(2, 8), groups=groups)
    elif kind == "trace":
        c.update(k=rng.randint(1, 128))
    elif kind == "triples":
        c.update(p=rng.choice([1.0, 0.5, 0.1]), samples=_log_uniform(rng, 1000, 1 << 25), hybrid=rng.random() < 0.5)
    elif kind == "stream":
        c.update(d=rng.choice([0.5, 1.0, 2.0]), samples=_log_uniform(rng, 1000, 1 << 24))
    elif kind == "serve":
        n = 1 << rng.randint(12, 18)  # the largest request
        c.update(graph="rmat", n=n, pairs=16 * n, requests=rng.randint(4, 48), lanes=rng.choice([1, 4]),
                 fuse_max_pairs=rng.choice([0, 262144]))
    return c


# ---- inputs ----------------------------------------------------------------


def _pairs(graph, n, count, seed):
    """(src, dst) int32 on the device; duplicates and loops as they fall."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    if graph == "chung-lu":  # endpoints drawn with probability ~ i ** (-1 / (beta - 1)), beta = 2.4
        w = torch.arange(1, n + 1, device=DEV, dtype=torch.float64).pow(-1.0 / 1.4).cumsum(0)
        ends = []
        for _ in range(2):
            x = torch.rand(count, generator=g, device=DEV, dtype=torch.float64) * w[-1]
            ends.append(torch.searchsorted(w, x).clamp_(max=n - 1))
    else:  # R-MAT (.57, .19, .19, .05); ids past an odd n wrap around
        u = torch.zeros(count, device=DEV, dtype=torch.int32)
        v = torch.zeros(count, device=DEV, dtype=torch.int32)
        for _ in range(max(1, (n - 1).bit_length())):
            r = torch.rand(count, generator=g, device=DEV)
            u.mul_(2).add_(r >= 0.76)
            v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        ends = [u.remainder_(n), v.remainder_(n)]
    perm = torch.randperm(n, generator=g, device=DEV)
    return [perm[e.long()].to(torch.int32) for e in ends]


def _requests(case, seed):
    """One burst: scale uniform in [10, log2 n], p in {1, .5, .1}, pairs in pinned host memory."""
    rs = np.random.RandomState(seed % (1 << 31))
    out = []
    for i in range(case["requests"]):
        n = 1 << rs.randint(10, case["n"].bit_length())
        src, dst = (t.cpu().pin_memory().numpy() for t in _pairs("rmat", n, 16 * n, seed + 1 + i))
        out.append((n, src, dst, SERVE_P[rs.randint(3)], i))
    return out


def prepare(case, seed):
    if case["kind"] == "serve":
        server = tc.Server(8 << 30, lanes=case["lanes"], fuse_max_pairs=case["fuse_max_pairs"])
        return dict(case=case, server=server, requests=_requests(case, seed))
    src, dst = _pairs(case["graph"], case["n"], case["pairs"], seed)
    if case["kind"] == "build":
        # col has room for every pair; what the graph's entries do not fill stays -1
        out = [torch.full((size,), -1, dtype=torch.int32, device=DEV)
               for size in (case["n"] + 1, 2 * case["pairs"], case["n"])]
        return dict(case=case, src=src, dst=dst, out=out)
    return dict(case=case, graph=tc.tc_build_csr(case["n"], src, dst), seed=seed)


# ---- one pass --------------------------------------------------------------


def _read_into(graph, row, col, deg):
    """The CSR into the caller's device tensors (the tc_graph_read entry point)."""
    import ctypes
    from paper_1011_0468_amd import _native
    ptrs = [ctypes.c_void_p(t.data_ptr()) for t in (row, col, deg)]
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    _native.check(_native.load().tc_graph_read(graph.handle, *ptrs, 1, stream))


def _fields(counts):
    return np.array([[c[k] for k in sorted(c)] for c in counts], dtype=np.int64)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "build":
        _read_into(tc.tc_build_csr(case["n"], state["src"], state["dst"]), *state["out"])
        return dict(zip(("row_ptr", "col", "deg"), state["out"]))
    if kind == "serve":
        server = state["server"]
        for n, src, dst, p, seed in state["requests"]:
            server.submit(seed, p, seed, n=n, src=src, dst=dst)
        res = sorted(server.drain(), key=lambda r: r["id"])
        return dict(status=np.array([r["status"] for r in res]), counts=_fields([r["counts"] for r in res]),
                    estimate=np.array([r["estimate"] for r in res]))
    g = state["graph"]
    if kind in ("count", "noalloc"):
        heavy = (case["heavy_num"], case["heavy_den"])
        if kind == "noalloc":
            counts, est = tc.tc_estimate_noalloc(g, case["p"], state["seed"], heavy=heavy)
        elif case["p"] == 1.0:
            counts = tc.tc_count_exact(g, heavy=heavy)
            est = float(counts["triangles"])
        else:
            per, ests, _ = tc.tc_estimate(g, case["p"], [state["seed"]], heavy=heavy)
            counts, est = per[0], ests[0]
        return dict(counts, estimate=est)
    if kind == "batch":
        seeds = range(state["seed"], state["seed"] + case["seeds"])
        per, ests, mom = tc.tc_estimate(g, case["p"], seeds, num_groups=case["groups"])
        return dict(counts=_fields(per), estimates=np.array(ests), median_of_means=mom)
    if kind == "trace":
        q, est = tc.tc_rp_trace(g, case["k"], state["seed"])
        return dict(q=q, estimate=est)
    if kind == "triples":
        return tc.tc_triple_estimate(g, case["p"], case["samples"], hybrid=case["hybrid"], sample_seed=state["seed"],
                                     triple_seed=state["seed"])
    return tc.tc_stream_estimate(g, case["d"], case["samples"], seed=state["seed"])


def work(case):
    """Bytes of one pass: each edge once from its list of either end (and its random partners where the
    method draws them), each vertex's row start, and the results; the additions of the trace as flops."""
    n, m, kind = case["n"], case["pairs"], case["kind"]
    graph = 8 * m + 4 * n  # both directions of every edge, row starts
    if kind == "build":
        return dict(bytes=8 * m + graph, flops=0)
    if kind == "trace":  # Y = A X in 32 bits written and read once
        return dict(bytes=graph + 8 * n * case["k"], flops=4 * m * case["k"])
    if kind in ("triples", "stream"):  # a draw reads the two ids of its pair
        return dict(bytes=graph + 8 * case["samples"], flops=0)
    if kind == "serve":  # pairs in, of about 2 n / log2(n / 512) * 16 a request
        return dict(bytes=int(8 * case["requests"] * 32 * n / max(1, n.bit_length() - 10)), flops=0)
    if kind == "batch":
        return dict(bytes=graph + int(case["seeds"] * case["p"] * 8 * m), flops=0)
    return dict(bytes=graph, flops=0)


# ---- the same in plain torch, in 64 bits -------------------------------------


def _simple(n, src, dst):
    """Row, column of every entry of the simple undirected graph, sorted."""
    a, b = src.to(DEV).long(), dst.to(DEV).long()
    keep = a != b
    key = torch.unique(torch.cat([a[keep] * n + b[keep], b[keep] * n + a[keep]]))
    return torch.div(key, n, rounding_mode="floor"), key % n


def _shift(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _mix64(z):
    z = (z ^ _shift(z, 30)) * -0x40A7B892E31B1A47
    z = (z ^ _shift(z, 27)) * -0x6B2FB644ECCEEE15
    return z ^ _shift(z, 31)


def _word(x):
    return torch.tensor((x & (2 ** 64 - 1)) - (2 ** 64 if x & (1 << 63) else 0), device=DEV)


def _sampled(row, col, p, seed):
    salt = _mix64(_word(seed ^ 0x54435F53414D504C))
    h = _mix64(_mix64((torch.minimum(row, col) << 32) | torch.maximum(row, col)) ^ salt)
    keep = _shift(h, 11) < int(p * 2 ** 53)
    return row[keep], col[keep]


def _triangles(n, row, col):
    """By listing the wedges at each edge's lower end, lists ordered by degree."""
    deg = torch.bincount(row, minlength=n)
    rank = torch.empty(n, dtype=torch.long, device=DEV)
    rank[torch.argsort(deg * n + torch.arange(n, device=DEV))] = torch.arange(n, device=DEV)
    a, b = rank[row], rank[col]
    keys = torch.sort(a[a < b] * n + b[a < b])[0]
    a, b = torch.div(keys, n, rounding_mode="floor"), keys % n
    end = torch.bincount(a, minlength=n).cumsum(0)
    after = end[a] - torch.arange(len(a), device=DEV) - 1  # partners of each edge behind it in its list
    total, at, cum = 0, 0, after.cumsum(0)
    while at < len(a):
        done = int(cum[at - 1]) if at else 0
        to = max(at + 1, int(torch.searchsorted(cum, done + (1 << 27))))
        cnt = after[at:to]
        first = torch.repeat_interleave(torch.arange(at, to, device=DEV), cnt)
        step = torch.arange(len(first), device=DEV) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
        want = b[first] * n + b[first + 1 + step]
        pos = torch.searchsorted(keys, want).clamp_(max=len(keys) - 1)
        total += int((keys[pos] == want).sum())
        at = to
    return total


def _counted(n, row, col, p, seed):
    if p < 1.0:
        row, col = _sampled(row, col, p, seed)
    t = _triangles(n, row, col) if len(row) else 0
    return t, len(row) // 2, t / (p * p * p)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "serve" or (kind == "batch" and case["seeds"] * case["pairs"] > 1 << 28):
        return None
    row, col = _simple(n, *_pairs(case["graph"], n, case["pairs"], seed))
    if kind == "build":
        start = torch.zeros(n + 1, dtype=torch.long, device=DEV)
        start[1:] = torch.bincount(row, minlength=n).cumsum(0)
        cols = torch.full((2 * case["pairs"],), -1, dtype=torch.int32, device=DEV)
        cols[:len(col)] = col.to(torch.int32)
        return dict(row_ptr=start.to(torch.int32), col=cols, deg=start.diff().to(torch.int32))
    if kind in ("count", "noalloc"):
        if case["pairs"] * min(1.0, 2 * case["p"]) > 3 << 23:
            return None
        t, m, est = _counted(n, row, col, case["p"], seed)
        return dict(triangles=t, m=m, estimate=est)
    if kind == "batch":
        ts = [_counted(n, row, col, case["p"], seed + i) for i in range(case["seeds"])]
        per = case["seeds"] // case["groups"]
        sums = sorted(sum(t for t, _, _ in ts[i * per:(i + 1) * per]) for i in range(case["groups"]))
        mid = (sums[(len(sums) - 1) // 2] + sums[len(sums) // 2]) / 2 / per / case["p"] ** 3
        return dict(counts=None, estimates=np.array([e for _, _, e in ts]), median_of_means=mid)
    if kind == "trace":
        salt = _mix64(_word(seed ^ 0x52505F5452414345))
        q = []
        for v in range(case["k"]):
            bits = _mix64(_mix64(((v >> 6) << 32) | torch.arange(n, device=DEV)) ^ salt)
            x = 1 - 2 * ((bits >> (v & 63)) & 1)
            pre = torch.zeros(n + 1, dtype=torch.long, device=DEV)
            start = torch.searchsorted(row, torch.arange(n + 1, device=DEV)) if v == 0 else start
            y = torch.cat([pre[:1], x[col].cumsum(0)])[start].diff()
            q.append(int((y[row] * y[col]).sum()))
        return dict(q=np.array(q), estimate=sum(q) / (6 * case["k"]))
    if kind == "stream":
        m = len(row) // 2
        return dict(m=m, draws1=math.ceil(case["d"] * math.sqrt(m) * math.log(n)) if m else 0)
    if case["p"] < 1.0:
        row, col = _sampled(row, col, case["p"], seed)
    return dict(m=len(row) // 2)
