"""GPU parity of edges_to_csr against the oracle (bit-exact rows, columns,
duplicate counts and degree histograms)."""
import numpy as np
import pytest

from paper_1003_3684_amd import workloads as wl

pytestmark = pytest.mark.gpu

FLAG_SETS = [0, 1, 2, 3]  # directed, symmetrized, simple, symmetrized+simple


def _gpu_csr(sfg, n, src_np, dst_np, flags, id_bytes):
    import torch
    dt = torch.int32 if id_bytes == 4 else torch.int64
    src = torch.as_tensor(np.asarray(src_np), dtype=dt).cuda()
    dst = torch.as_tensor(np.asarray(dst_np), dtype=dt).cuda()
    rp, col, hist, dups = sfg.edges_to_csr(n, src, dst, flags=flags)
    torch.cuda.synchronize()
    assert sfg.device_error() == 0
    return rp.cpu().numpy(), col.cpu().numpy(), hist.cpu().numpy(), int(dups.item())


def _check(sfg, orc, n, src, dst, flags, id_bytes):
    rp, col, hist, dups = _gpu_csr(sfg, n, src, dst, flags, id_bytes)
    orp, ocol, odups = orc.edges_to_csr(n, src, dst, symmetrize=bool(flags & 1), simple=bool(flags & 2))
    _, ohist = orc.degree_histogram(n, src, dst)
    np.testing.assert_array_equal(rp.astype(np.uint64), orp)
    kept = int(orp[-1])
    np.testing.assert_array_equal(col[:kept].astype(np.int64), ocol)
    assert dups == odups
    np.testing.assert_array_equal(hist.astype(np.uint64), ohist)


@pytest.mark.parametrize("flags", FLAG_SETS)
def test_csr_kron_k20(sfg, orc, flags):
    """The 2^24-edge Kronecker graph: directed CSR with about 691 k repeated edges."""
    c = wl.KRON_K20
    src, dst = orc.kron_sample(c["n0"], c["initiator"], c["k"], c["num_edges"], c["seed"])
    _check(sfg, orc, c["n0"] ** c["k"], src, dst, flags, 4)


@pytest.mark.parametrize("flags", FLAG_SETS)
def test_csr_pba_small(sfg, orc, flags):
    c = wl.PBA_SMALL
    src, dst = orc.pba_generate(c["n"], c["m"], c["num_parts"], c["p_inter"], c["seed"])
    _check(sfg, orc, c["n"], src, dst, flags, 4)


@pytest.mark.parametrize("trial", range(16))
def test_csr_random(sfg, orc, trial):
    rng = np.random.default_rng(500 + trial)
    n = int(rng.choice([1, 2, 3, 17, 1000, 65536, 65537, 1 << 20, (1 << 24) + 3]))
    E = int(rng.choice([0, 1, 5, 8191, 8192, 8193, 100_000, 300_001]))
    id_bytes = 8 if trial % 2 else 4
    if rng.uniform() < 0.5:  # skewed ids, many repeats and self-loops
        src = np.minimum(rng.zipf(1.5, size=E) - 1, n - 1)
        dst = np.minimum(rng.zipf(1.8, size=E) - 1, n - 1)
    else:
        src = rng.integers(0, n, size=E)
        dst = rng.integers(0, n, size=E)
    flags = int(rng.integers(0, 4))
    _check(sfg, orc, n, src.astype(np.int64), dst.astype(np.int64), flags, id_bytes)


def test_csr_wide_ids(sfg):
    """n = 2^31 - 1 (62 live key bits): columns match a lexicographic sort and
    row starts match binary searches at sampled rows (row_ptr stays on the GPU)."""
    import torch
    rng = np.random.default_rng(3)
    n = (1 << 31) - 1
    E = 50_000
    src = np.concatenate([rng.integers(n - 1000, n, size=E - 10), np.full(10, n - 1)])
    dst = rng.integers(0, n, size=E)
    s = torch.as_tensor(src, dtype=torch.int64).cuda()
    d = torch.as_tensor(dst, dtype=torch.int64).cuda()
    rp, col, hist, dups = sfg.edges_to_csr(n, s, d, flags=0)
    torch.cuda.synchronize()
    order = np.lexsort((dst, src))
    np.testing.assert_array_equal(col.cpu().numpy(), dst[order])
    ss = src[order]
    rows = np.concatenate([[0, 1, n - 1001, n - 1, n], rng.integers(n - 1100, n, size=200)])
    got = rp[torch.as_tensor(rows).cuda()].cpu().numpy()
    np.testing.assert_array_equal(got, np.searchsorted(ss, rows, side="left"))
    key = src * n + dst
    assert int(dups.item()) == E - len(np.unique(key))
    del rp
    torch.cuda.empty_cache()


def test_csr_all_loops_and_empty(sfg, orc):
    n = 10
    src = np.array([3, 3, 3, 7, 7], np.int64)
    dst = src.copy()
    for flags in FLAG_SETS:
        _check(sfg, orc, n, src, dst, flags, 4)
    for flags in FLAG_SETS:
        _check(sfg, orc, n, np.zeros(0, np.int64), np.zeros(0, np.int64), flags, 4)


@pytest.mark.parametrize("order", ["ascending", "descending", "blocks"])
@pytest.mark.parametrize("flags", [0, 1])
def test_csr_sorted_inputs(sfg, orc, order, flags):
    """Inputs already ordered by source (or in reverse, or in sorted blocks):
    each digit value of the last pass sits in a few tiles only, so most
    tiles' runs follow a run of an earlier, non-adjacent tile or of another
    digit -- the cases the last pass settles after the sort."""
    rng = np.random.default_rng({"ascending": 1, "descending": 2, "blocks": 3}[order] + 10 * flags)
    n, E = (1 << 20) + 5, 200_003
    src = rng.integers(0, n, size=E)
    dst = rng.integers(0, n, size=E)
    if order == "ascending":
        src = np.sort(src)
    elif order == "descending":
        src = np.sort(src)[::-1].copy()
    else:
        src = np.concatenate([np.sort(b) for b in np.array_split(src, 7)])
    dst[::97] = src[::97]  # some self-loops
    dst[1::89] = dst[0:-1:89][: len(dst[1::89])]  # some repeated pairs next to each other
    src[1::89] = src[0:-1:89][: len(src[1::89])]
    for ib in (4, 8):
        _check(sfg, orc, n, src, dst, flags, ib)


def test_entry_count_limit(sfg):
    """More than 2^34 entries (edges, doubled when symmetrized) is ERANGE,
    found before any buffer is touched: with one workgroup per tile a
    dispatch's work-item count stays below 2^32."""
    import torch
    lib = sfg.load()
    t = torch.zeros(64, dtype=torch.int64, device="cuda")
    p = t.data_ptr()
    for num_edges, flags in (((1 << 34) + 1, 0), ((1 << 33) + 1, sfg.CSR_SYMMETRIZE)):
        rc = lib.edges_to_csr(1000, num_edges, p, p, 8, flags, p, p, None, None, p, 1 << 62, None)
        assert rc == sfg.SFG_ERANGE, (num_edges, flags, rc)
    torch.cuda.synchronize()
    assert int(t.abs().sum().item()) == 0


@pytest.mark.parametrize("flags", FLAG_SETS)
@pytest.mark.parametrize("n,E", [(16 * 4096 - 1, 20_000), (16 * 4096, 20_000), (5 * 4096 - 7, 9), (1 << 22, 100),
                                 ((1 << 22) + 5, 20_000), (40_000, 0)])
def test_csr_row_fill_branches(sfg, orc, flags, n, E):
    """Both sides of the rules of the row fill: its own chunks' next marks (up
    to 16 chunks of 4,096 rows), the chunk scan, and the arrays one after the
    other (more than 2^19 rows per tile of entries); long empty stretches."""
    rng = np.random.default_rng(n + E)
    src, dst = rng.integers(0, n, size=E), rng.integers(n // 3, n // 2, size=E)
    src[: E // 2] = src[: E // 2] // 7
    _check(sfg, orc, n, src, dst, flags, 4)


def test_csr_histogram_pointer_of_8_byte_alignment(sfg, orc):
    """degree_hist32 and num_duplicates need only the alignment of their type."""
    import ctypes as C
    import torch
    rng = np.random.default_rng(8)
    n, E = 3000, 10_000
    src, dst = rng.integers(0, n, size=E), rng.integers(0, n, size=E)
    s, d = (torch.as_tensor(x, dtype=torch.int32).cuda() for x in (src, dst))
    buf = torch.full((40,), -1, dtype=torch.int64, device="cuda")
    rp, col = torch.empty(n + 1, dtype=torch.int64, device="cuda"), torch.empty(E, dtype=torch.int32, device="cuda")
    ws = sfg.workspace(sfg.edges_to_csr_workspace_bytes(n, E, 4, 0))
    p = lambda t, off=0: C.c_void_p(t.data_ptr() + off)
    rc = sfg.load().edges_to_csr(n, E, p(s), p(d), 4, 0, p(rp), p(col), p(buf, 8), p(buf, 8 * 35), p(ws), ws.numel(),
                                 C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    _, hist = orc.degree_histogram(n, src, dst)
    _, _, dups = orc.edges_to_csr(n, src, dst)
    np.testing.assert_array_equal(got[1:33].astype(np.uint64), hist)
    assert got[35] == dups and got[0] == -1 and (got[33:35] == -1).all() and (got[36:] == -1).all()


@pytest.mark.parametrize("id_bytes,n", [(4, 3_000), (8, 300_000)])
@pytest.mark.parametrize("E", [2047, 2048, 2049, 64 * 2048, 64 * 2048 + 1])
def test_csr_short_tiles(sfg, orc, E, id_bytes, n):
    """Directed lists around the short tiles' edges and around the longest
    list sorted in them, with 4- and 8-byte keys."""
    rng = np.random.default_rng(E)
    src = np.minimum(rng.zipf(1.6, size=E) - 1, n - 1)
    _check(sfg, orc, n, src, rng.integers(0, n, size=E), 0, id_bytes)


@pytest.mark.parametrize("id_bytes", [4, 8])
@pytest.mark.parametrize("E", [1, 63, 65, 1023, 1025, 8191, 8192, 8193, 16_385, 40_000])
@pytest.mark.parametrize("shape", ["runs", "one pair", "loops", "one vertex", "sparse"])
def test_csr_simple_finish_tiles(sfg, orc, shape, E, id_bytes):
    """Runs of equal entries, self-loops and row starts across the lanes, waves and
    tiles of the compacting finish, for lists that end inside each of them."""
    import torch
    rng = np.random.default_rng(E + id_bytes)
    n = {"runs": 40, "one pair": 5, "loops": 300, "one vertex": 1, "sparse": 70_001}[shape]
    src = rng.integers(0, n, E)
    dst = rng.integers(0, n, E)
    if shape == "one pair":
        src[:], dst[:] = 3, 1
    if shape == "loops":
        dst = np.where(rng.uniform(size=E) < 0.9, src, dst)
    t = torch.int32 if id_bytes == 4 else torch.int64
    rp, col, hist, dups = sfg.edges_to_csr(n, torch.tensor(src, dtype=t, device="cuda"),
                                           torch.tensor(dst, dtype=t, device="cuda"), flags=sfg.CSR_SIMPLE)
    torch.cuda.synchronize()
    assert sfg.device_error() == 0
    orp, ocol, odups = orc.edges_to_csr(n, src, dst, symmetrize=False, simple=True)
    np.testing.assert_array_equal(rp.cpu().numpy().astype(np.uint64), orp.astype(np.uint64))
    np.testing.assert_array_equal(col[:int(orp[-1])].cpu().numpy().astype(np.int64), ocol)
    assert int(dups.item()) == odups


@pytest.mark.parametrize("flags", FLAG_SETS)
@pytest.mark.parametrize("n", [1, 3, 1022, 1023, 1024, 4095, 16_384, 65_537, 131_071, 131_072])
@pytest.mark.parametrize("rows", ["first", "last", "sparse"])
def test_csr_row_fill_short_chunks(sfg, orc, rows, n, flags):
    """Chunks of 1,024 rows (up to 2^17 - 1 vertices) and the chunk scan above:
    lists whose rows lie at one end, so that the next marked row is far or there
    is none, or a few rows apart."""
    rng = np.random.default_rng(n)
    E = 700
    src = rng.integers(0, min(n, 5), size=E) if rows != "sparse" else rng.integers(0, n, size=E)
    src = n - 1 - src if rows == "last" else src
    dst = rng.integers(0, min(n, 9), size=E)
    _check(sfg, orc, n, src, dst, flags, 4)


@pytest.mark.parametrize("n,flags", [(200, 0), (70_000, 0), (70_000, 1), (70_000, 3)])
def test_row_starts_over_the_edge_list(sfg, n, flags):
    """row_ptr in the memory of src: the list is read before any row start is written."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n + flags)
    E = n + 4_321
    src = torch.randint(0, n, (E,), device="cuda", generator=g)
    dst = torch.randint(0, n, (E,), device="cuda", generator=g)
    want = sfg.edges_to_csr(n, src, dst, flags=flags)
    got = sfg.edges_to_csr(n, src, dst, flags=flags, row_ptr=src[:n + 1])
    kept = int(want[0][n])
    assert torch.equal(got[0], want[0]) and torch.equal(got[1][:kept], want[1][:kept])
    assert torch.equal(got[2], want[2]) and torch.equal(got[3], want[3])


@pytest.mark.parametrize("id_bytes,n", [(4, 3_000), (8, 300_000)])
@pytest.mark.parametrize("E", [28 * 2048, 30 * 2048 - 1, 30 * 2048, 30 * 2048 + 1, 31 * 3072 - 1, 31 * 3072, 31 * 3072 + 1])
def test_csr_longest_short_tile_lists(sfg, orc, E, id_bytes, n):
    """Directed and symmetrized lists on both sides of the most entries that are
    sorted in short tiles, whose look-back words are the narrow ones."""
    rng = np.random.default_rng(E)
    src = np.minimum(rng.zipf(1.6, size=E) - 1, n - 1)
    dst = rng.integers(0, n, size=E)
    _check(sfg, orc, n, src, dst, 0, id_bytes)
    _check(sfg, orc, n, src[:E // 2], dst[:E // 2], 3, id_bytes)


def test_short_lists_in_a_workspace_made_for_a_longer_one(sfg):
    """One buffer, sized for the longest list, serves every shorter one."""
    import torch
    n, longest = 5_000, 142_784
    ws = sfg.workspace(sfg.edges_to_csr_workspace_bytes(n, longest, 4, 0))
    src = torch.randint(0, n, (longest,), device="cuda", dtype=torch.int32)
    dst = torch.randint(0, n, (longest,), device="cuda", dtype=torch.int32)
    for E in (longest, 131_073, 131_072, 61_441, 61_440, 100, 0):
        want = sfg.edges_to_csr(n, src[:E], dst[:E])
        got = sfg.edges_to_csr(n, src[:E], dst[:E], ws=ws)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1][:E], want[1][:E]) and torch.equal(got[2], want[2])


@pytest.mark.parametrize("n", [5_000_011, 8_700_000, 17_400_000, 20_000_003])
@pytest.mark.parametrize("E", [0, 3, 2_500])
def test_csr_few_entries_over_many_rows(sfg, n, E):
    """Row starts, columns and histogram where the row fill's chunk scans are longer
    than the rest of the workspace (the arrays are then filled one after the
    other), and where they just fit, with one and with two arrays beside row_ptr."""
    import torch
    rng = np.random.default_rng(n + E)
    src, dst = rng.integers(0, n, E), rng.integers(0, n, E)
    if E:
        src[:2], dst[:2] = (0, n - 1), (n - 1, n - 1)
    for flags in FLAG_SETS:
        rp, col, hist, _ = _gpu_csr(sfg, n, src, dst, flags, 4)
        u, v = (np.concatenate([src, dst]), np.concatenate([dst, src])) if flags & 1 else (src, dst)
        key = np.sort(u * n + v)
        if flags & 2:
            key = np.unique(key[key // n != key % n])
        want = np.zeros(n + 1, np.int64)
        np.add.at(want, key // n + 1, 1)
        np.testing.assert_array_equal(rp, np.cumsum(want))
        np.testing.assert_array_equal(col[:len(key)], key % n)
        deg = np.bincount(np.concatenate([src, dst]), minlength=n)
        want = np.bincount(np.where(deg > 0, np.floor(np.log2(np.maximum(deg, 1))) + 1, 0).astype(np.int64), minlength=32)
        np.testing.assert_array_equal(hist, want)


@pytest.mark.parametrize("n", [17, 40, 191])
@pytest.mark.parametrize("E", [1, 10, 100, 600])
def test_csr_without_a_histogram_in_the_queried_workspace(sfg, orc, n, E):
    import torch
    rng = np.random.default_rng(n + E)
    src, dst = rng.integers(0, n, E), rng.integers(0, n, E)
    rp, col, _, dups = sfg.edges_to_csr(n, torch.tensor(src).cuda(), torch.tensor(dst).cuda(), want_hist=False)
    orp, ocol, odups = orc.edges_to_csr(n, src, dst)
    np.testing.assert_array_equal(rp.cpu().numpy().astype(np.uint64), orp)
    np.testing.assert_array_equal(col.cpu().numpy(), ocol)
    assert int(dups.item()) == odups
