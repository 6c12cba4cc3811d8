"""GPU parity of graph_stats against the oracle: the degree histogram and the
closed-wedge count bit for bit, the exponent within 1e-9 relative (binary64
sums in a different order)."""
import math

import numpy as np
import pytest

from paper_1003_3684_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(sfg, orc, n, src_np, dst_np, samples, seed, gid, id_bytes=4):
    import torch
    dt = torch.int32 if id_bytes == 4 else torch.int64
    src = torch.as_tensor(np.asarray(src_np), dtype=dt).cuda()
    dst = torch.as_tensor(np.asarray(dst_np), dtype=dt).cuda()
    hist, gamma, closed = sfg.graph_stats(n, src, dst, num_samples=samples, seed=seed, graph_id=gid)
    torch.cuda.synchronize()
    assert sfg.device_error() == 0
    ohist, ogamma, oclosed = orc.graph_stats(n, src_np, dst_np, samples, seed, gid)
    np.testing.assert_array_equal(hist.cpu().numpy().astype(np.uint64), ohist)
    assert int(closed.item()) == oclosed
    g = float(gamma.item())
    if math.isnan(ogamma):
        assert math.isnan(g)
    else:
        assert abs(g - ogamma) <= 1e-9 * abs(ogamma), (g, ogamma)


def test_stats_pba_small(sfg, orc):
    c = wl.PBA_SMALL
    src, dst = orc.pba_generate(c["n"], c["m"], c["num_parts"], c["p_inter"], c["seed"])
    _check(sfg, orc, c["n"], src, dst, 10_000, 17, 4)


def test_stats_kron(sfg, orc):
    W = [[0.57, 0.19], [0.19, 0.05]]
    src, dst = orc.kron_sample(2, W, 16, 1 << 20, 3, 9)
    _check(sfg, orc, 1 << 16, src, dst, 10_000, 17, 9)


@pytest.mark.parametrize("trial", range(8))
def test_stats_random(sfg, orc, trial):
    rng = np.random.default_rng(3000 + trial)
    n = int(rng.choice([3, 50, 1000, 70_000]))
    E = int(rng.choice([0, 1, 10, 5000, 200_000]))
    src = np.minimum(rng.zipf(1.6, size=E) - 1, n - 1)
    dst = rng.integers(0, n, size=E)
    _check(sfg, orc, n, src, dst, int(rng.choice([0, 1, 777, 10_000])), int(rng.integers(0, 2 ** 62)),
           int(rng.integers(0, 1 << 24)), 8 if trial % 2 else 4)


def test_stats_no_wedge(sfg, orc):
    # a single edge and a self-loop: no wedge anywhere
    _check(sfg, orc, 5, np.array([0, 3]), np.array([1, 3]), 100, 1, 0)


@pytest.mark.parametrize("samples", [0, 500])
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 1024 * 4096, 1024 * 4096 + 1])
def test_stats_chunk_edges(sfg, orc, n, samples):
    """Vertex counts around a chunk and around the 1,024 chunk sums that the
    workgroups add up themselves; the hub sits in the last chunk, and one list has
    no wedge."""
    rng = np.random.default_rng(n + samples)
    E = min(3 * n, 40_000)
    src = np.where(rng.uniform(size=E) < 0.3, n - 1, rng.integers(0, n, size=E))
    dst = rng.integers(0, n, size=E)
    _check(sfg, orc, n, src, dst, samples, 5, 3)
    _check(sfg, orc, n, src[:1], dst[:1], samples, 5, 3, 8)


@pytest.mark.parametrize("samples", [1, 15, 16, 17, 65_535, 65_536, 65_537, 70_001])
def test_stats_sample_lanes(sfg, orc, samples):
    """Sample counts around a wavefront's groups of lanes and around the number
    from which a sample takes one lane, over rows of every length."""
    rng = np.random.default_rng(samples)
    n, E = 20_000, 60_000
    src = np.minimum(rng.zipf(1.5, size=E) - 1, n - 1)
    dst = np.minimum(rng.zipf(1.3, size=E) - 1, n - 1)
    _check(sfg, orc, n, src, dst, samples, 11, 6, 8 if samples % 2 else 4)


@pytest.mark.parametrize("samples", [32_767, 32_768, 32_769])
def test_stats_sample_lanes_at_their_line(sfg, orc, samples):
    """The last sample counts at 16 lanes each and the first at one (on 256 CUs)."""
    rng = np.random.default_rng(samples)
    n, E = 20_000, 60_000
    src = np.minimum(rng.zipf(1.5, size=E) - 1, n - 1)
    dst = np.minimum(rng.zipf(1.3, size=E) - 1, n - 1)
    _check(sfg, orc, n, src, dst, samples, 11, 6, 8 if samples % 2 else 4)
