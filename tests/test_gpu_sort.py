"""The sort's launch shapes, by what they decide: groups of four points on a wide lattice,
in shuffled input order, so that the labels are known without a search (a group's id is
the rank of its smallest input index). Sizes lie at the edges of a tile, of the tile sizes
and of the inputs sorted in one launch; the spacing of the lattice decides the width of
DenseBox's keys (10: 32 bits, 400: 64 bits at the sizes below)."""
import numpy as np
import pytest

from tests.test_gpu_parity import dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def lattice_groups(n, d, spacing, seed):
    rng = np.random.default_rng(seed)
    groups = -(-n // 4)
    side = int(np.ceil(groups ** (1.0 / d)))
    g = rng.permutation(np.arange(n) // 4)
    at = np.stack([g // side**k % side for k in range(d)], axis=1) * float(spacing)
    pts = (at + rng.uniform(0.0, 0.25, size=(n, d))).astype(np.float32)
    _, first, inverse = np.unique(g, return_index=True, return_inverse=True)
    want = np.argsort(np.argsort(first))[inverse]
    size = np.bincount(g)[g]
    return pts, want, size


@pytest.mark.parametrize("algo", ["fdbscan", "densebox"])
@pytest.mark.parametrize("d,spacing", [(2, 10), (3, 400)])
@pytest.mark.parametrize("n", [2, 5, 1024, 1025, 32768, 32769, 131072, 131073, 262144, 262145, 524288, 524289])
def test_sorted_groups(dev, algo, d, spacing, n):  # noqa: F811
    pts, want, size = lattice_groups(n, d, spacing, n + d)
    labels, core, _ = run_gpu(dev, pts, 1.0, 2, algo)
    # the last group of an odd size may be a lone point: noise, and no id of its own
    lone = size < 2
    ids = np.unique(want[~lone])
    want = np.where(lone, -1, np.searchsorted(ids, want))
    assert np.array_equal(labels, want)
    assert np.array_equal(core.astype(bool), ~lone)
