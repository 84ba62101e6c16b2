"""Border points whose neighbours were joined by walks of several XCDs at once: every XCD
has to read the same final labels afterwards. Which stores meet depends on timing, so each
scene is clustered many times (labels were wrong in more than half of the calls when walks
shortened chains with plain stores). Labels equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _say, dev  # noqa: F401

pytestmark = pytest.mark.gpu


def clumps(n, d, k, sigma, side, seed):
    rng = np.random.default_rng(seed)
    at, pts, inside = rng.uniform(0, side, (k, d)), rng.uniform(0, side, (n, d)), rng.random(n) < 0.8
    pts[inside] = at[rng.integers(0, k, inside.sum())] + sigma * rng.standard_normal((inside.sum(), d))
    return pts.astype(np.float32)


@pytest.mark.parametrize("algo", ["fdbscan", "densebox"])
@pytest.mark.parametrize("d,n,min_pts", [(2, 500000, 100), (2, 500000, 140), (2, 500000, 200), (3, 300000, 40)])
def test_border_labels_of_repeated_calls(dev, algo, d, n, min_pts):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    pts = clumps(n, d, 50, 3.0, 100, 2)
    ref, ref_core, ref_k = oracle.dbscan(pts, 1.0, min_pts)
    _say(f"[gpu] repeated calls: {algo} d={d} n={n} minPts={min_pts}")
    t, want = torch.from_numpy(pts).to(dev), torch.from_numpy(ref.astype(np.int32)).to(dev)
    want_core = torch.from_numpy(ref_core.astype(bool)).to(dev)
    off = []
    for _ in range(25):
        lab, core, k = fdb.dbscan(t, 1.0, min_pts, algo=algo)
        assert k == ref_k and bool((core == want_core).all())
        off.append(int((lab != want).sum()))
    assert off == [0] * 25
