"""DenseBox where cells that are not dense hold many points (a large minPts): once the core
pass is done, a cell's core points are one set, and walks pass over cells of their own set.
Alone, with the first claim, and in batches; minPts on both sides of where sets are made, and
cells of just under, at and over the points that they are made for. Labels equal the
oracle's; and such calls take not many times what one with a small minPts takes."""
import time

import numpy as np
import pytest

import oracle
from tests.helpers import assert_tolerance_mode
from tests.test_gpu_parity import _say, assert_exact, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def lattice(d, per_cell, seed, n=9000):
    """About `per_cell` points a cell of side 1/sqrt(d), more towards one corner."""
    rng = np.random.default_rng(seed)
    side = (n / per_cell) ** (1 / d) / np.sqrt(d)
    return (side * rng.random((n, d)) ** 1.2).astype(np.float32)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("per_cell", [6, 8, 30])
@pytest.mark.parametrize("min_pts", [16, 17, 40, 120])
def test_cells_below_min_pts(dev, d, per_cell, min_pts):  # noqa: F811
    pts = lattice(d, per_cell, 11 * d + per_cell)
    ref = assert_exact(dev, pts, 1.0, min_pts, "densebox")
    lab, core, _ = run_gpu(dev, pts, 1.0, min_pts, "densebox", border="first")
    assert_tolerance_mode(pts, 1.0, lab, core, ref[0], ref[1], oracle.check_border)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("mp", [[2, 16, 5, 10], [2, 17, 60, 150], [200, 40, 2, 90]])
def test_batch(dev, d, mp):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    clouds = [lattice(d, 5 + 12 * k, k + d, n=1500 + 700 * k) - np.float32(3 * k) for k in range(len(mp))]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    _say(f"[gpu] batch of cells d={d} minPts={mp}")
    for border in ("canonical", "first"):
        lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), torch.from_numpy(off),
                                          torch.ones(len(mp)), torch.tensor(mp, dtype=torch.int32), algo="densebox",
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


@pytest.mark.parametrize("d,ball,min_pts", [(3, 1500, 300)])
def test_time_with_a_large_min_pts(dev, d, ball, min_pts):  # noqa: F811
    # evenly spread points, all core; minPts 10 makes every cell dense
    import torch
    import paper_2103_05162_amd as fdb
    _say(f"[gpu] cells of a large minPts d={d}")
    n = 200000
    side = (n * (4 / 3 * np.pi if d == 3 else np.pi) / ball) ** (1 / d)
    t = torch.from_numpy(np.random.default_rng(3).uniform(0, side, (n, d)).astype(np.float32)).to(dev)
    med = []
    for mp in (10, min_pts):
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, _, k = fdb.dbscan(t, 1.0, mp, algo="densebox")
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        assert k == 1
        med.append(float(np.median(times[1:])))
    _say(f"[gpu]   minPts 10 {1e6 * med[0]:.0f} us, {min_pts} {1e6 * med[1]:.0f} us")
    assert med[1] < 10.0 * med[0]  # (6 times; 15 times with every point looked up)
