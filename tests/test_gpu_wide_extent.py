"""DenseBox in a scene whose extent is beyond the largest float: the grid has no cells for
it, so neighbours are searched through the hierarchy, which takes no more than 40 times
what the scene takes without its two far points (a search that meets every point took
190 times that). Labels are those of the scene alone."""
import time

import numpy as np
import pytest

from tests.test_gpu_parity import _say, dev  # noqa: F401

pytestmark = pytest.mark.gpu


def call(dev, pts, algo, min_pts):
    import torch
    import paper_2103_05162_amd as fdb
    t = torch.from_numpy(pts).to(dev)
    times = []
    for _ in range(6):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        lab, core, k = fdb.dbscan(t, 1.0, min_pts, algo=algo)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    return lab.cpu().numpy(), core.cpu().numpy(), k, float(np.median(times[1:]))


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("axes", [1, 3])
@pytest.mark.parametrize("algo", ["densebox", "auto"])
@pytest.mark.parametrize("min_pts", [2, 5])
def test_two_points_at_the_ends(dev, d, axes, algo, min_pts):  # noqa: F811
    _say(f"[gpu] widest extent d={d} axes={axes} {algo} minPts={min_pts}")
    rng = np.random.default_rng(7)
    n = 60000
    at = rng.uniform(0, 100, size=(20, d))
    pts = rng.uniform(0, 100, size=(n, d))
    inside = rng.random(n) < 0.8
    pts[inside] = at[rng.integers(0, 20, inside.sum())] + 2.0 * rng.standard_normal((inside.sum(), d))
    pts = np.sort(pts, axis=0).astype(np.float32)  # in input order along the axes
    far = np.full((2, d), 50.0, np.float32)
    far[0, :axes], far[1, :axes] = -3e38, 3e38
    if axes < d:  # (the other coordinates: away from every point)
        far[:, axes:] = 1000.0
    ref = call(dev, pts, algo, min_pts)
    lab, core, k, t = call(dev, np.concatenate([pts, far]), algo, min_pts)
    assert k == ref[2] and np.array_equal(lab[:n], ref[0]) and np.array_equal(core[:n], ref[1])
    assert (lab[n:] < 0).all() and not core[n:].any()
    _say(f"[gpu]   {1e6 * t:.0f} us, without them {1e6 * ref[3]:.0f} us")
    assert t < 40.0 * ref[3]
