"""DenseBox's compactions at the edges of their tiles (4096 points) and of the number of
tiles whose counts are added up where they are used (512): groups of four points on a
lattice in shuffled order, which are dense cells or points of several cells, so that
the labels are known without a search."""
import numpy as np
import pytest

from tests.test_gpu_parity import dev, run_gpu  # noqa: F401
from tests.test_gpu_sort import lattice_groups

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("n", [4095, 4096, 4097, 8193, 100000, 512 * 4096, 512 * 4096 + 1])
def test_tiles(dev, d, n):  # noqa: F811
    pts, want, size = lattice_groups(n, d, 10, n + d)
    labels, core, k = run_gpu(dev, pts, 1.0, 2, "densebox")
    lone = size < 2
    ids = np.unique(want[~lone])
    assert k == ids.size
    assert np.array_equal(labels, np.where(lone, -1, np.searchsorted(ids, want)))
    assert np.array_equal(core.astype(bool), ~lone)
