"""DenseBox where a few cells hold thousands of points and are not dense: a scene so wide that
the rounding of cell coordinates puts points past their cell's edges, or a minPts above what
they hold. Labels equal the oracle's, and a wide scene with most of its points in a few cells
takes less than three times what FDbscan takes (five when each cell was stepped through by one
lane)."""
import time

import numpy as np
import pytest

import oracle
from tests.helpers import assert_tolerance_mode
from tests.test_gpu_parity import _say, assert_exact, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def scales(d, n, seed, decades=3.0):
    """Points of log-uniform distance from the middle."""
    r, s = np.random.default_rng(seed), np.random.default_rng(seed + 1)
    return (10.0 ** r.uniform(-3, decades, (n, 1)) * s.standard_normal((n, d))).astype(np.float32)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("n,min_pts", [(12000, 5), (12000, 700), (6000, 2), (20000, 9000), (700, 120)])
def test_labels(dev, d, n, min_pts):  # noqa: F811
    pts = scales(d, n, n + d, decades=3.0 if d == 2 else 1.5)
    ref = assert_exact(dev, pts, 1.0, min_pts, "densebox")
    if min_pts > 2:
        lab, core, _ = run_gpu(dev, pts, 1.0, min_pts, "densebox", border="first")
        assert_tolerance_mode(pts, 1.0, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("size", [63, 64, 65, 127, 128, 129, 500])
def test_cells_of_equal_size(dev, size):  # noqa: F811
    # every cell holds `size` points, all of one or of many cells in a wavefront's box
    rng = np.random.default_rng(size)
    at = np.stack(np.meshgrid(np.arange(9), np.arange(9)), -1).reshape(-1, 2) * 0.70
    pts = (at[:, None, :] + rng.uniform(0.01, 0.6, (81, size, 2))).reshape(-1, 2).astype(np.float32)
    for min_pts in (size + 1, 3 * size, 12 * size):
        assert_exact(dev, pts, 1.0, min_pts, "densebox")


def test_time(dev):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    _say("[gpu] heavy cells in a wide scene")
    t = torch.from_numpy(scales(2, 500000, 3)).to(dev)
    med, out = {}, {}
    for algo in ("fdbscan", "densebox"):
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            out[algo] = fdb.dbscan(t, 1.0, 5, algo=algo)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        med[algo] = float(np.median(times[1:]))
    assert out["fdbscan"][2] == out["densebox"][2]
    assert bool((out["fdbscan"][0] == out["densebox"][0]).all()) and bool((out["fdbscan"][1] == out["densebox"][1]).all())
    _say(f"[gpu]   FDbscan {1e6 * med['fdbscan']:.0f} us, DenseBox {1e6 * med['densebox']:.0f} us")
    assert med["densebox"] < 3.0 * med["fdbscan"]
