"""Sampled shortest-path statistics (Results, Table 2) on the GPU against the
oracle's breadth-first searches and against closed forms: sums of distances,
reachable pairs and the largest distance must agree exactly."""
import numpy as np
import pytest

from paper_1003_3684_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _undirected_csr(n, pairs):
    a = np.array(pairs, np.int64).reshape(-1, 2)
    u = np.concatenate([a[:, 0], a[:, 1]])
    v = np.concatenate([a[:, 1], a[:, 0]])
    keep = u != v
    key = np.unique(u[keep] * n + v[keep])
    u, v = key // n, key % n
    rp = np.zeros(n + 1, np.uint64)
    np.add.at(rp, u + 1, 1)
    return np.cumsum(rp).astype(np.uint64), v.astype(np.int64)


def _gpu(sfg, n, rp, col, sources, id_bytes=4):
    import torch
    rp_d = torch.tensor(rp.astype(np.int64), device="cuda")
    col_d = torch.tensor(col.astype(np.int32 if id_bytes == 4 else np.int64), device="cuda")
    if col_d.numel() == 0:
        col_d = torch.zeros(1, dtype=col_d.dtype, device="cuda")
    out = sfg.path_stats(n, rp_d, col_d, sources)
    torch.cuda.synchronize()
    return tuple(int(x) for x in out.cpu().numpy())


@pytest.mark.parametrize("id_bytes", [4, 8])
def test_closed_forms(sfg, orc, id_bytes):
    n = 50
    rp, col = _undirected_csr(n, [(i, i + 1) for i in range(n - 1)])
    assert _gpu(sfg, n, rp, col, [0], id_bytes) == (n * (n - 1) // 2, n - 1, n - 1)
    # star with a heavy centre (degree above the one-lane limit)
    n = 1001
    rp, col = _undirected_csr(n, [(0, i) for i in range(1, n)])
    assert _gpu(sfg, n, rp, col, [0, 7], id_bytes) == ((n - 1) + 1 + 2 * (n - 2), 2 * (n - 1), 2)
    d = 7
    n = 1 << d
    rp, col = _undirected_csr(n, [(v, v ^ (1 << b)) for v in range(n) for b in range(d)])
    srcs = list(range(0, n, 3))  # 43 sources
    assert _gpu(sfg, n, rp, col, srcs, id_bytes) == (len(srcs) * d * (1 << (d - 1)), len(srcs) * (n - 1), d)
    rp, col = _undirected_csr(6, [(0, 1), (1, 2), (3, 4)])
    assert _gpu(sfg, 6, rp, col, [0, 3, 5, 5], id_bytes) == (4, 3, 2)


@pytest.mark.parametrize("kind", ["pba", "kron"])
def test_generated_graphs_match_oracle(sfg, orc, kind):
    import torch
    if kind == "pba":
        n, E = 6000, 6000 * 3
        src, dst = sfg.pba_generate(n, 3, 8, 0.2, seed=5)
    else:
        k = 12
        n, E = 1 << k, 16 << k
        src, dst = sfg.kron_generate(2, [[0.57, 0.19], [0.19, 0.05]], k, E, seed=9)
    rp, col, _, _ = sfg.edges_to_csr(n, src, dst, flags=sfg.CSR_SYMMETRIZE | sfg.CSR_SIMPLE)
    torch.cuda.synchronize()
    kept = int(rp[-1])
    sources = np.random.default_rng(2).integers(0, n, 150)  # three groups, the last partial
    out = sfg.path_stats(n, rp, col[:max(kept, 1)], sources)
    torch.cuda.synchronize()
    got = tuple(int(x) for x in out.cpu().numpy())
    want = orc.path_stats(n, rp.cpu().numpy().astype(np.uint64), col[:kept].cpu().numpy().astype(np.int64), sources)
    assert got == want
    assert want[1] > 0 and 1 <= want[2] < 64


def test_errors(sfg):
    import torch
    from paper_1003_3684_amd.native import SfgenError
    rp, col = _undirected_csr(4, [(0, 1), (2, 3)])
    rp_d = torch.tensor(rp.astype(np.int64), device="cuda")
    col_d = torch.tensor(col.astype(np.int32), device="cuda")
    with pytest.raises(SfgenError):
        sfg.path_stats(4, rp_d, col_d, [4])
    with pytest.raises(SfgenError):
        sfg.path_stats(4, rp_d, col_d, [0], ws=sfg.workspace(8))
    assert _gpu(sfg, 4, rp, col, []) == (0, 0, 0)


@pytest.mark.parametrize("hub", [16, 17, 255, 256, 257, 4095, 4096, 4097, 8200])
def test_degree_classes_match_oracle(sfg, orc, hub):
    """Hubs on both sides of the degrees above which more lanes, a wavefront
    and several wavefronts sweep a vertex; a path behind each, so that the search runs
    over several batches of levels; two groups of sources, the second ragged
    and with repeats."""
    rng = np.random.default_rng(hub)
    n = hub + 90
    pairs = [(0, i) for i in range(1, hub + 1)]          # vertex 0: degree hub (+ 1 below)
    pairs += [(hub + i, hub + i + 1) for i in range(40)]  # a path that starts at a leaf
    pairs += [(n - 2, n - 1)]                             # a component of its own
    extra = rng.integers(1, hub + 1, size=(hub, 2))
    rp, col = _undirected_csr(n, pairs + [tuple(p) for p in extra])
    srcs = np.concatenate([rng.integers(0, n, 70), [0, hub + 40, n - 1, n - 1]])
    exp = orc.path_stats(n, rp, col, srcs)
    for id_bytes in (4, 8):
        assert _gpu(sfg, n, rp, col, srcs, id_bytes) == tuple(int(x) for x in exp)


@pytest.mark.parametrize("n,deg,tail", [(64, 4200, 0), (40, 4097, 11), (300, 17, 11), (5000, 40, 11)])
def test_listed_degrees_match_oracle(sfg, orc, n, deg, tail):
    """Multigraphs whose vertices are all listed: nearly all above the huge degree
    (at 64 vertices more than its list holds), or all of a middle degree; a tail of
    a few vertices, so that most of the search finds nothing left in them."""
    rng = np.random.default_rng(n + deg)
    u = np.repeat(np.arange(n), (deg + 1) // 2)
    v = (u + 1 + rng.integers(0, n - 1, len(u))) % n
    path = np.arange(n - 1, n + tail)  # behind the last vertex
    u, v = np.concatenate([u, path[:-1]]), np.concatenate([v, path[1:]])
    u, v = np.concatenate([u, v]), np.concatenate([v, u])
    order = np.argsort(u, kind="stable")
    total = n + tail
    rp = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=total))]).astype(np.uint64)
    col = v[order].astype(np.int64)
    srcs = rng.integers(0, total, 70)
    exp = orc.path_stats(total, rp, col, srcs)
    for id_bytes in (4, 8):
        assert _gpu(sfg, total, rp, col, srcs, id_bytes) == tuple(int(x) for x in exp)


@pytest.mark.parametrize("id_bytes", [4, 8])
def test_listed_only_by_others_matches_oracle(sfg, orc, id_bytes):
    """Rows that list a source whose own row is empty: a level ORs the words of
    the neighbours a row lists, so the source reaches those rows (a breadth-first
    search of the transposed graph)."""
    rng = np.random.default_rng(11)
    n = 400
    pairs = [(v, 0) for v in range(1, 60)]                    # row 0 is empty
    pairs += [(v, int(rng.integers(1, 60))) for v in range(60, 300)]
    pairs += [(v, v - 1) for v in range(301, n)]              # a chain read from its head, whose row is empty
    a = np.array(sorted(pairs), np.int64)
    t = a[np.argsort(a[:, 1], kind="stable")][:, ::-1]
    rp, trp = (np.concatenate([[0], np.cumsum(np.bincount(x[:, 0], minlength=n))]).astype(np.uint64) for x in (a, t))
    for srcs in ([0], [300], [0, 300, 7, 0]):
        exp = orc.path_stats(n, trp, t[:, 1], np.array(srcs))
        assert exp[1] > 50
        assert _gpu(sfg, n, rp, a[:, 1], srcs, id_bytes) == tuple(int(x) for x in exp)


@pytest.mark.parametrize("n", [2**18 - 1, 2**18, 2**18 + 1, 2**19, 2**19 + 33, 2**20 + 77, 2**22 - 5])
@pytest.mark.parametrize("id_bytes", [4, 8])
def test_coarse_bitmap_sizes_match_oracle(sfg, orc, n, id_bytes):
    """Vertices on both sides of the sizes at which a bit of the coarse bitmap stands
    for 1, 2, 4, 8 and 16 of them.  Half of them hang on a few hubs (more than 4,096
    edges) and on each other, so that the frontier fills, passes an eighth of the
    vertices and empties again; a path of 40 behind the last, some cycles far from
    the hubs, and idle vertices between; two groups of sources."""
    import torch
    rng = np.random.default_rng(n)
    core = n // 2
    u = np.concatenate([rng.integers(0, 6, core), rng.integers(0, core, core // 2), rng.integers(6, 300, core // 8)])
    v = np.concatenate([np.arange(core), rng.integers(0, core, core // 2), rng.integers(0, core, core // 8)])
    tail = np.arange(n - 41, n - 1)
    ring = np.arange(core + 1000, core + 1200)
    u = np.concatenate([u, tail, [core - 1], ring, [ring[-1]]])
    v = np.concatenate([v, tail + 1, [n - 41], ring + 1, [ring[0]]])
    src, dst = torch.tensor(u).cuda(), torch.tensor(v).cuda()
    rp, col, _, _ = sfg.edges_to_csr(n, src, dst, flags=sfg.CSR_SYMMETRIZE | sfg.CSR_SIMPLE)
    kept = int(rp[-1])
    col = col[:kept].to(torch.int32) if id_bytes == 4 else col[:kept]
    sources = np.concatenate([rng.integers(0, core, 3), [n - 1, int(ring[7]), n - 50, 2]])
    if id_bytes == 4:  # a second group, in which most sources are near
        sources = np.concatenate([np.resize(sources[:4], 64), sources[4:]])
    out = sfg.path_stats(n, rp, col, sources)
    got = tuple(int(x) for x in out.cpu().numpy())
    uniq, times = np.unique(sources, return_counts=True)
    parts = [orc.path_stats(n, rp.cpu().numpy().astype(np.uint64), col.cpu().numpy().astype(np.int64), np.array([s])) for s in uniq]
    want = (sum(int(p[0]) * int(t) for p, t in zip(parts, times)), sum(int(p[1]) * int(t) for p, t in zip(parts, times)),
            max(int(p[2]) for p in parts))
    assert got == want
    assert want[2] >= 42


def test_more_vertices_than_32_bit_ids(sfg):
    """Above 2^32 vertices (nearly all idle): 64-bit lists, no bitmaps.  A hub shared by
    several wavefronts, one swept by a wavefront, one of 40 edges and a path across
    2^32; 68 sources, some repeated, against a search over the few rows with entries."""
    import collections
    import torch
    n = (1 << 32) + 70_001
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 175 << 30:
        pytest.skip("needs 175 GiB of GPU memory")
    hub, leaf, path = n - 1, n - 60_000, n - 40_000
    pairs = [(hub, leaf + i) for i in range(5_000)] + [(17, v) for v in range((1 << 32) - 300, (1 << 32) + 300)]
    pairs += [(23, v) for v in range(100, 140)] + [(path + i, path + i + 1) for i in range(12)]
    pairs += [(leaf, 17), (23, 17), (path, 100)]
    a = np.array(pairs, np.int64)
    a = np.concatenate([a, a[:, ::-1]])
    a = a[np.lexsort((a[:, 1], a[:, 0]))]
    ids, counts = np.unique(a[:, 0], return_counts=True)
    starts = np.cumsum(counts)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    for v, end, at in zip(ids, np.append(ids[1:], n), starts):
        rp[int(v) + 1:int(end) + 1] = int(at)
    neighbours = collections.defaultdict(list)
    for u, v in a.tolist():
        neighbours[u].append(v)

    def search(s):
        dist, queue = {s: 0}, collections.deque([s])
        while queue:
            u = queue.popleft()
            for v in neighbours[u]:
                if v not in dist:
                    dist[v] = dist[u] + 1
                    queue.append(v)
        return sum(dist.values()), len(dist) - 1, max(dist.values())

    sources = [hub, 17, path + 10, 23, 50, leaf + 7] + [leaf + 1] * 62
    found = [search(s) for s in sources]
    out = sfg.path_stats(n, rp, torch.tensor(a[:, 1], device="cuda"), sources)
    assert tuple(out.tolist()) == (sum(f[0] for f in found), sum(f[1] for f in found), max(f[2] for f in found))
    del rp, out
    torch.cuda.empty_cache()
