"""DenseBox's neighbour search through the grid: grids one cell, one brick and one super
wide and a cell to either side of that on each axis, points on cell boundaries, and
the scenes that go through the hierarchy instead (a far outlier makes the grid too
wide for the table), alone and in batches. Labels equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.helpers import assert_tolerance_mode
from tests.test_gpu_parity import _say, assert_exact, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def scene(d, cells, n, seed, eps=0.125):
    """n points over `cells` grid cells per axis (side eps/sqrt(d)), a third of them in clumps."""
    rng = np.random.default_rng(seed)
    side = cells * eps / np.sqrt(d)
    pts = rng.uniform(0.0, side, size=(n, d))
    c = rng.uniform(0.0, side, size=(3, d))
    k = n // 3
    pts[:k] = c[rng.integers(0, 3, k)] + 0.3 * eps * rng.standard_normal((k, d))
    return np.clip(pts, 0.0, side).astype(np.float32), float(np.float32(eps))


# bricks are 4 (3D) or 8 (2D) cells wide, supers 16 or 64
EDGES = [(3, c) for c in (1, 3, 4, 5, 15, 16, 17, 33)] + [(2, c) for c in (1, 7, 8, 9, 63, 64, 65, 129)]


@pytest.mark.parametrize("d,cells", EDGES)
@pytest.mark.parametrize("min_pts", [2, 5])
def test_grid_edges(dev, d, cells, min_pts):  # noqa: F811
    pts, eps = scene(d, cells, 4097, 7 * cells + d)
    assert_exact(dev, pts, eps, min_pts, "densebox")


@pytest.mark.parametrize("d", [2, 3])
def test_points_on_cell_boundaries(dev, d):  # noqa: F811
    # multiples of half a cell side, rounded to float: neighbours at exactly eps and cells decided by rounding
    rng = np.random.default_rng(d)
    eps = 0.1
    pts = (rng.integers(0, 40, size=(6000, d)) * (0.5 * eps / np.sqrt(d))).astype(np.float32)
    pts = np.unique(pts, axis=0)
    for min_pts in (2, 9, 40):
        assert_exact(dev, pts, float(np.float32(eps)), min_pts, "densebox")


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("min_pts", [1, 2, 5])
def test_outlier_goes_through_the_hierarchy(dev, d, min_pts):  # noqa: F811
    pts, eps = scene(d, 24, 3000, 11 + d)
    pts[-1] = 3000.0 if d == 3 else 50000.0  # more supers than two a point
    ref = oracle.dbscan(pts, eps, min_pts)
    assert_exact(dev, pts, eps, min_pts, "densebox", ref=ref)
    if min_pts > 2:
        lab, core, _ = run_gpu(dev, pts, eps, min_pts, "densebox", border="first")
        assert_tolerance_mode(pts, eps, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("n", [70, 3000, 40000])
def test_first_claim_through_the_grid(dev, d, n):  # noqa: F811
    pts, eps = scene(d, 20, n, 5 * d)
    ref = oracle.dbscan(pts, eps, 6)
    lab, core, _ = run_gpu(dev, pts, eps, 6, "densebox", border="first")
    assert_tolerance_mode(pts, eps, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("wide", [False, True])
def test_batch_grids(dev, d, wide):  # noqa: F811
    """Clouds of other extents, sizes and eps in one batch; `wide`: one of them too wide for its grid."""
    import torch
    import paper_2103_05162_amd as fdb
    clouds, eps = [], []
    for k, (cells, n) in enumerate([(1, 1), (3, 700), (17, 2500), (40, 900), (5, 64), (66, 1500)]):
        p, e = scene(d, cells, n, 31 + k, eps=0.05 * (k + 1))
        clouds.append(p - np.float32(0.7 * k))
        eps.append(e)
    if wide:
        clouds[2][0] = 1.0e4
    mp = [1, 2, 5, 3, 4, 6]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    _say(f"[gpu] batch d={d} wide={wide}")
    lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), torch.from_numpy(off),
                                      torch.tensor(eps, dtype=torch.float32), torch.tensor(mp, dtype=torch.int32),
                                      algo="densebox")
    torch.cuda.synchronize()
    lab, core, k = lab.cpu().numpy(), core.cpu().numpy(), k.cpu().numpy()
    for c, p in enumerate(clouds):
        rl, rc, rk = oracle.dbscan(p, eps[c], mp[c])
        s = slice(off[c], off[c + 1])
        assert k[c] == rk and np.array_equal(core[s], rc) and np.array_equal(lab[s], rl), f"cloud {c}"
