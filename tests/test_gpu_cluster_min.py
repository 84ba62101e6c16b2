"""Each cluster's smallest input index (which orders the canonical ids), taken a
wavefront of 256 points at a time: sizes at the edges of that tile, with one root
per tile, a few, and as many as points (minPts 1 without neighbours), and one
cluster spread among others along the curve. Labels are whole numbers: equal to
the oracle's."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import assert_exact, dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", ["fdbscan", "densebox"])
@pytest.mark.parametrize("min_pts", [1, 3])
@pytest.mark.parametrize("n", [255, 256, 257, 1023, 1025])
def test_cluster_minimum_at_tile_edges(dev, n, min_pts, algo):  # noqa: F811
    pts = np.random.default_rng(n).uniform(0.0, 1.0, size=(n, 2)).astype(np.float32)
    for eps in (1e-5, 0.6 / np.sqrt(n), 1.1 / np.sqrt(n), 2.0):  # alone, scattered, percolating, one cluster
        e = float(np.float32(eps))
        assert_exact(dev, pts, e, min_pts, algo, ref=oracle.dbscan(pts, e, min_pts))
