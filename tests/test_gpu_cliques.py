"""FDbscan's cliques (subtrees whose points are pairwise within eps): clumps of sizes
around the least clique, the least that searches by itself and a wavefront, minPts around
the clump's size, clumps that just touch or just miss each other, and clumps whose box
has a diagonal of eps or a rounding more. Alone and in batches; labels equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.helpers import assert_tolerance_mode
from tests.test_gpu_parity import _say, assert_exact, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

EPS = float(np.float32(0.25))


def clumps(d, size, seed, noise=200):
    """Clumps of `size` points in a box of diagonal eps/2, about eps apart in a chain, and some noise."""
    rng = np.random.default_rng(seed)
    at = np.cumsum(rng.uniform(0.5, 0.8, size=(24, d)) * EPS, axis=0)
    pts = [c + rng.uniform(0, 0.5 * EPS / np.sqrt(d), size=(size, d)) for c in at]
    pts.append(rng.uniform(0, at.max() + EPS, size=(noise, d)))
    p = np.concatenate(pts).astype(np.float32)
    return p[rng.permutation(len(p))]


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("size", [1, 3, 4, 5, 7, 8, 15, 16, 17, 63, 64, 65, 200])
def test_clumps(dev, d, size):  # noqa: F811
    pts = clumps(d, size, 10 * size + d)
    for min_pts in sorted({1, 2, 3, max(1, size - 1), size, size + 1, 2 * size}):
        ref = assert_exact(dev, pts, EPS, min_pts, "fdbscan")
        if min_pts > 2:
            lab, core, _ = run_gpu(dev, pts, EPS, min_pts, "fdbscan", border="first")
            assert_tolerance_mode(pts, EPS, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("grow", [-1, 0, 1])
def test_box_of_diagonal_eps(dev, d, grow):  # noqa: F811
    # points at the corners of a box whose diagonal is eps, a float more or a float less
    side = np.float32(3.0), np.float32(4.0), np.float32(0.0)
    eps = 5.0
    b = np.nextafter(side[1], np.float32(4.0 + grow)) if grow else side[1]
    corners = np.array([[x, y, 0.0][:d] for x in (0, side[0]) for y in (0, b)], np.float32)
    pts = np.concatenate([corners] * 9 + [corners + np.float32(40.0)] * 3).astype(np.float32)
    for min_pts in (2, 5, 18, 27, 28, 36, 37):
        assert_exact(dev, pts, eps, min_pts, "fdbscan")


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("axes", [1, 2, 3])
@pytest.mark.parametrize("far", [1.0e4, 1.0e9])
def test_far_point(dev, d, axes, far):  # noqa: F811
    # one point far out on some axes: the curve's cells there are wider than eps
    pts = clumps(d, 20, 17 * d + axes, noise=3000)
    pts[5, :axes] = far  # (all axes: more than a key holds)
    for min_pts in (2, 10):
        assert_exact(dev, pts, EPS, min_pts, "fdbscan")


@pytest.mark.parametrize("d", [2, 3])
def test_batch_of_clumps(dev, d):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    sizes = [1, 4, 16, 33, 5, 90, 64]
    clouds = [clumps(d, s, s + d, noise=50 + s) - np.float32(0.3 * k) for k, s in enumerate(sizes)]
    eps = [EPS * (1.0 + 0.25 * (k % 3)) for k in range(len(sizes))]
    mp = [2, 3, 17, 30, 1, 20, 64]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    _say(f"[gpu] batch of clumps d={d}")
    lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), torch.from_numpy(off),
                                      torch.tensor(eps, dtype=torch.float32), torch.tensor(mp, dtype=torch.int32),
                                      algo="fdbscan")
    torch.cuda.synchronize()
    lab, core, k = lab.cpu().numpy(), core.cpu().numpy(), k.cpu().numpy()
    for c, p in enumerate(clouds):
        rl, rc, rk = oracle.dbscan(p, float(np.float32(eps[c])), mp[c])
        s = slice(off[c], off[c + 1])
        assert k[c] == rk and np.array_equal(core[s], rc) and np.array_equal(lab[s], rl), f"cloud {c}"
