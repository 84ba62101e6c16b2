"""FDbscan over scenes too wide for its keys on every axis: bodies of dense clumps far apart,
of equal and unequal size, also interleaved in input order, and many of them. Each body's
labels are those of a call for it alone (ids shifted by its place), and the call takes no
more than four times what the bodies' own calls take together: where the curve's cells are
wide against a body's clumps, it takes tens of times that."""
import time

import numpy as np
import pytest

from tests.test_gpu_parity import _say, assert_exact, dev  # noqa: F401

pytestmark = pytest.mark.gpu

EPS = 0.002


def body(seed, n, at):
    """Clumps of about 13,000 points (width 0.0005) over a thin background, its corner at `at`."""
    rng = np.random.default_rng(seed)
    side = (n / 8388608) ** (1 / 3)
    centers = rng.uniform(0, side, size=(max(1, round(n / 16777)), 3))
    p = rng.uniform(0, side, size=(n, 3))
    inside = rng.random(n) < 0.8
    p[inside] = centers[rng.integers(0, len(centers), inside.sum())] + 5e-4 * rng.standard_normal((inside.sum(), 3))
    return (p + at).astype(np.float32)


def call(dev, pts, min_pts):
    import torch
    import paper_2103_05162_amd as fdb
    t = torch.from_numpy(pts).to(dev)
    times = []
    for _ in range(6):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        lab, core, k = fdb.dbscan(t, EPS, min_pts, algo="fdbscan")
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    return lab.cpu().numpy(), core.cpu().numpy(), k, float(np.median(times[1:]))


CASES = {
    "two": [(1000000, 0.0), (300000, 4000.0)],
    "small_second": [(1000000, 4000.0), (50000, 0.0)],
    "interleaved": [(600000, 0.0), (600000, 4000.0)],
    "ten": [(100000, 400.0 * k * k) for k in range(10)],
}


@pytest.mark.parametrize("min_pts", [2, 10])
@pytest.mark.parametrize("case", list(CASES))
def test_far_bodies(dev, case, min_pts):  # noqa: F811
    _say(f"[gpu] far bodies: {case} minPts={min_pts}")
    bodies = [body(k + 1, n, at) for k, (n, at) in enumerate(CASES[case])]
    alone = [call(dev, p, min_pts) for p in bodies]
    want, first = [], 0
    for lab, _, k, _ in alone:
        want.append(np.where(lab >= 0, lab + first, -1))
        first += k
    pts, want, core = np.concatenate(bodies), np.concatenate(want), np.concatenate([a[1] for a in alone])
    if case == "interleaved":  # one point of each in turn; ids go by the smallest input index
        turn = np.arange(len(pts)).reshape(2, -1).T.ravel()
        pts, want, core = pts[turn], want[turn], core[turn]
        ids, at = np.unique(want[core], return_index=True)
        new = np.empty(ids.max() + 1, np.int64)
        new[ids[np.argsort(at)]] = np.arange(ids.size)
        far = np.unique(want[want >= 0])
        assert np.array_equal(far, ids)  # (a border point's cluster has core points)
        renamed = np.where(want >= 0, new[np.maximum(want, 0)], -1)
    else:
        renamed = want
    lab, got_core, k, t = call(dev, pts, min_pts)
    assert k == first and np.array_equal(got_core, core)
    # a border point between two clusters takes the smaller id, which interleaving may change
    same = core | (want < 0) if case == "interleaved" else np.ones(len(pts), bool)
    assert np.array_equal(lab[same], renamed[same])
    assert np.array_equal(lab < 0, renamed < 0)
    together = sum(a[3] for a in alone)
    _say(f"[gpu]   {1e6 * t:.0f} us, the bodies alone {1e6 * together:.0f} us")
    assert t < 4.0 * together


@pytest.mark.parametrize("n", [5, 60, 1023, 1025, 3000])
def test_few_points_far_apart(dev, n):  # noqa: F811
    # fewer points than the curve's sample has, and just more: bodies of five points each
    rng = np.random.default_rng(n)
    at = rng.uniform(0, 1e7, size=(-(-n // 5), 3))
    pts = (at.repeat(5, axis=0)[:n] + rng.uniform(0, 4.0, size=(n, 3))).astype(np.float32)
    for min_pts in (2, 4):
        assert_exact(dev, pts, 2.5, min_pts, "fdbscan")
