"""FDbscan where a box of diagonal eps holds fewer than minPts points but an eps-ball many
(the box's core points are one set once the core pass is done), and cliques of more points
than one search takes. Labels equal the oracle's; and such calls take not many times what
their like take: before boxes of core points were joined, every pair was tested, and a
clique of any size searched as one."""
import time

import numpy as np
import pytest

import oracle
from tests.helpers import assert_tolerance_mode
from tests.test_gpu_parity import _say, assert_exact, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def spread(d, n, ball, seed):
    """n points, `ball` of them expected within 1 of a point, denser towards one corner."""
    rng = np.random.default_rng(seed)
    side = (n * (4 / 3 * np.pi if d == 3 else np.pi) / ball) ** (1 / d)
    return (side * rng.random((n, d)) ** 1.3).astype(np.float32)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("min_pts", [5, 9, 13, 40, 130, 300])
def test_boxes_below_min_pts(dev, d, min_pts):  # noqa: F811
    pts = spread(d, 12000, 250, 3 * d + min_pts)
    ref = assert_exact(dev, pts, 1.0, min_pts, "fdbscan")
    lab, core, _ = run_gpu(dev, pts, 1.0, min_pts, "fdbscan", border="first")
    assert_tolerance_mode(pts, 1.0, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
def test_boxes_of_a_batch(dev, d):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    mp = [2, 5, 30, 60, 200, 13]
    clouds = [spread(d, 2000 + 500 * k, 40 + 60 * k, 7 * k + d) for k in range(len(mp))]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    _say(f"[gpu] batch of boxes d={d}")
    for border in ("canonical", "first"):
        lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), torch.from_numpy(off),
                                          torch.ones(len(mp)), torch.tensor(mp, dtype=torch.int32), algo="fdbscan",
                                          border=border)
        torch.cuda.synchronize()
        lab, core, k = lab.cpu().numpy(), core.cpu().numpy(), k.cpu().numpy()
        for c, p in enumerate(clouds):
            rl, rc, rk = oracle.dbscan(p, 1.0, mp[c])
            s = slice(off[c], off[c + 1])
            if border == "canonical":
                assert k[c] == rk and np.array_equal(core[s], rc) and np.array_equal(lab[s], rl), c
            else:
                assert_tolerance_mode(p, 1.0, lab[s], core[s], rl, rc, oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("size", [511, 512, 513, 1025, 3000])
@pytest.mark.parametrize("single", [False, True])
def test_large_cliques(dev, d, size, single):  # noqa: F811
    # a chain of bodies within eps each, some within eps of the next; `single`: one point of a
    # body stands apart from the others, which are all alike (a leaf beside the rest)
    rng = np.random.default_rng(size + d)
    pts = []
    for b in range(5):
        p = rng.uniform(0, 0.5, (size, d))
        if single:
            p[:] = p[0]
            p[1] += 0.2
        pts.append(p + b * rng.uniform(0.6, 1.1))
    pts.append(rng.uniform(-1, 5, (300, d)))
    pts = np.concatenate(pts).astype(np.float32)
    pts = pts[rng.permutation(len(pts))]
    for min_pts in (2, 5, 513, 600, 2 * size):
        ref = assert_exact(dev, pts, 1.0, min_pts, "fdbscan")
        if min_pts > 2:
            lab, core, _ = run_gpu(dev, pts, 1.0, min_pts, "fdbscan", border="first")
            assert_tolerance_mode(pts, 1.0, lab, core, ref[0], ref[1], oracle.check_border)


def timed(dev, pts, min_pts):
    import torch
    import paper_2103_05162_amd as fdb
    t = torch.from_numpy(pts).to(dev)
    times = []
    for _ in range(6):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        lab, core, k = fdb.dbscan(t, 1.0, min_pts, algo="fdbscan")
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    return lab.cpu().numpy(), k, float(np.median(times[1:]))


@pytest.mark.parametrize("d", [2, 3])
def test_bodies_that_nearly_touch(dev, d):  # noqa: F811
    # balls of diameter 0.56, each a clique; boxes within 1 of each other but no pair
    _say(f"[gpu] bodies that nearly touch d={d}")
    rng = np.random.default_rng(5)
    n = 30000
    v = rng.standard_normal((2 * n, d))
    v *= 0.28 * rng.random((2 * n, 1)) ** (1 / d) / np.linalg.norm(v, axis=1, keepdims=True)
    v[n:] += 1.57 / np.sqrt(d)
    v = v.astype(np.float32)
    alone = timed(dev, v[:n], 10)[2] + timed(dev, v[n:], 10)[2]
    lab, k, t = timed(dev, v, 10)
    assert k == 2 and (lab[:n] == 0).all() and (lab[n:] == 1).all()
    _say(f"[gpu]   {1e6 * t:.0f} us, the bodies alone {1e6 * alone:.0f} us")
    assert t < 25.0 * alone  # (2 to 3 times; 500 times and more with one search a clique)


@pytest.mark.parametrize("d,ball,few,many", [(3, 1700, 10, 100), (2, 4000, 100, 1000)])
def test_min_pts_above_a_box(dev, d, ball, few, many):  # noqa: F811
    # evenly spread points: all core either way, in boxes of at least `few` but never `many`
    _say(f"[gpu] minPts above a box d={d}")
    n = 200000
    side = (n * (4 / 3 * np.pi if d == 3 else np.pi) / ball) ** (1 / d)
    pts = np.random.default_rng(3).uniform(0, side, (n, d)).astype(np.float32)
    times = []
    for min_pts in (few, many):
        lab, k, t = timed(dev, pts, min_pts)
        assert k == 1
        times.append(t)
    _say(f"[gpu]   minPts {few} {1e6 * times[0]:.0f} us, {many} {1e6 * times[1]:.0f} us")
    assert times[1] < 10.0 * times[0]  # (3 and 6 times; 16 and 18 times with every pair tested)
