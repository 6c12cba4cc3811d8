"""Randomized PK by temporary seed modification (PK section): the GPU's
level-synchronous expansion equals the oracle's meta-edge stack entry for
entry, including edge order, and reduces to enumerate mode without changes."""
import numpy as np
import pytest

from paper_1003_3684_amd import workloads as wl

pytestmark = pytest.mark.gpu

FIG2 = wl.FIG2_SEED.astype(np.float32)
SEED3 = np.array([[1, 1, 0], [0, 1, 1], [1, 0, 0]], np.float32)
ONES8 = np.ones((8, 8), np.float32)


@pytest.mark.parametrize("seed_m,k,p_add,p_del,id_bytes", [
    (FIG2, 1, 0.3, 0.3, 4),       # the seed itself
    (FIG2, 4, 0.0, 0.0, 4),       # the deterministic power
    (FIG2, 6, 0.05, 0.1, 4),      # ~1.5 M edges, several scan blocks
    (SEED3, 9, 0.2, 0.3, 8),      # 64-bit ids
    (SEED3, 5, 1.0, 1.0, 4),      # every cell flipped: seed (x) complement^4
    (SEED3, 4, 0.0, 1.0, 4),      # everything deleted below the first level
    # ~58 children per meta-edge: a workgroup's children overflow its LDS
    # staging area and are written directly
    (ONES8, 3, 0.0, 0.1, 4),
    (ONES8, 3, 0.0, 0.1, 8),
])
def test_matches_oracle(sfg, orc, seed_m, k, p_add, p_del, id_bytes):
    import torch
    n0 = seed_m.shape[0]
    cap = 4_000_000
    src, dst = sfg.kron_perturbed(n0, seed_m, k, p_add, p_del, cap, seed=17, graph_id=2, id_bytes=id_bytes)
    torch.cuda.synchronize()
    os_, od = orc.kron_perturbed(seed_m, k, p_add, p_del, 17, 2, cap=cap)
    np.testing.assert_array_equal(src.cpu().numpy().astype(np.int64), os_)
    np.testing.assert_array_equal(dst.cpu().numpy().astype(np.int64), od)


@pytest.mark.parametrize("n0,cells,k,p_add,p_del", [
    (2, 1, 12, 0.4, 0.1), (3, 4, 7, 0.1, 0.2), (4, 16, 5, 0.0, 0.3), (5, 1, 2, 0.0, 0.0),
    (6, 9, 4, 0.1, 0.0),      # more than 32 cells: 64-bit masks
    (7, 49, 3, 0.0, 0.5), (8, 3, 4, 0.02, 0.0),
    (8, 64, 3, 0.0, 0.0),     # the most children of a round: 256 x 64
])
def test_granules_and_cell_masks_match_oracle(sfg, orc, n0, cells, k, p_add, p_del):
    import torch
    m = np.zeros(n0 * n0, np.float32)
    m[np.random.default_rng(n0 * 100 + cells).permutation(n0 * n0)[:cells]] = 1
    m = m.reshape(n0, n0)
    cap = 2_000_000
    os_, od = orc.kron_perturbed(m, k, p_add, p_del, 23, 1, cap=cap)
    for capacity in (max(len(os_), cells), cap):  # (no level is larger than the last one allows, or is stopped below)
        try:
            src, dst = sfg.kron_perturbed(n0, m, k, p_add, p_del, capacity, seed=23, graph_id=1)
        except Exception:
            assert capacity != cap and p_del > 0  # a level before the last was larger
            continue
        torch.cuda.synchronize()
        np.testing.assert_array_equal(src.cpu().numpy().astype(np.int64), os_)
        np.testing.assert_array_equal(dst.cpu().numpy().astype(np.int64), od)


def test_level_too_large_names_its_iteration(sfg):
    from paper_1003_3684_amd.native import SfgenError
    with pytest.raises(SfgenError, match=r"iteration 3 has 1331 edges, capacity is 1330"):
        sfg.kron_perturbed(5, FIG2, 6, 0.0, 0.0, 1330)


def test_no_change_equals_enumerate(sfg):
    import torch
    a = sfg.kron_perturbed(5, FIG2, 5, 0.0, 0.0, 11 ** 5, seed=3)
    b = sfg.kron_generate(5, FIG2, 5, 11 ** 5, mode=sfg.KRON_ENUMERATE)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_capacity_error(sfg):
    from paper_1003_3684_amd.native import SfgenError
    with pytest.raises(SfgenError):
        sfg.kron_perturbed(5, FIG2, 4, 0.0, 0.0, 11 ** 4 - 1)
    with pytest.raises(SfgenError):
        sfg.kron_perturbed(9, np.ones((9, 9), np.float32), 2, 0.0, 0.0, 100)


@pytest.mark.parametrize("n0,cells,k,p_add,p_del", [(2, 1, 12, 0.4, 0.1), (3, 4, 7, 0.1, 0.2), (4, 16, 5, 0.0, 0.3),
                                                    (7, 49, 3, 0.0, 0.5), (3, 3, 9, 0.0, 0.6), (3, 3, 9, 0.0, 1.0)])
def test_capacity_decides_by_the_first_level_above_it(sfg, orc, n0, cells, k, p_add, p_del):
    """The first iteration above the capacity is named, with its size, and no output is
    touched; a capacity that every level fits gives the edges.  The sizes are the oracle's,
    of the powers by fewer levels."""
    import ctypes
    import re
    import torch
    m = np.zeros(n0 * n0, np.float32)
    m[np.random.default_rng(n0 * 100 + cells).permutation(n0 * n0)[:cells]] = 1
    m = m.reshape(n0, n0)
    edges = [orc.kron_perturbed(m, it, p_add, p_del, 23, 1, cap=3_000_000) for it in range(1, k + 1)]
    sizes = [len(e[0]) for e in edges]
    lib = sfg.load()
    for capacity in sorted({cells, sizes[-1], max(sizes) - 1, max(sizes), max(sizes) + 7, max(sizes[:-1])} - {0}):
        if capacity < cells:
            continue
        src = torch.full((capacity,), -7, dtype=torch.int32, device="cuda")
        dst, count = src.clone(), torch.full((1,), -7, dtype=torch.int64, device="cuda")
        ws = sfg.workspace(lib.kron_perturbed_workspace_bytes(capacity))
        p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
        rc = lib.kron_perturbed(n0, m.ctypes.data_as(ctypes.c_void_p), k, p_add, p_del, 23, 1, 4, capacity, p(src), p(dst),
                                p(count), p(ws), ws.numel(), None)
        above = [it for it in range(2, k + 1) if sizes[it - 1] > capacity]
        if above:
            assert rc == sfg.SFG_ENOSPACE
            assert re.search(f"iteration {above[0]} has {sizes[above[0] - 1]} edges, capacity is {capacity}$",
                             lib.sfg_last_error().decode())
            assert int(count) == -7 and bool((src == -7).all()) and bool((dst == -7).all())
        else:
            assert rc == 0 and int(count) == sizes[-1]
            np.testing.assert_array_equal(src[:sizes[-1]].cpu().numpy(), edges[-1][0])
            np.testing.assert_array_equal(dst[:sizes[-1]].cpu().numpy(), edges[-1][1])
