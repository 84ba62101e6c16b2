"""An eps whose square leaves the normal range of fp32: the test s <= fl32(eps * eps) then
passes pairs farther apart than eps (both sides 0, or both infinite), or by how denormals
round. Also eps on both sides of where DenseBox's grid stops serving (2^-60 and 2^63).
Alone and as one cloud of a batch; labels equal the oracle's."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _say, assert_exact, dev  # noqa: F401

pytestmark = pytest.mark.gpu

EPS = [1e-30, 1e-23, 3e-22, 3e-21, 1e-20, 2e-19, 2.0**-61, 2.0**-60, 1e-17, 9e18, 2.0**63, 1.2e19, 1.8e19, 1.9e19,
       3e19, 1e25]


def scene(d, eps, seed):
    """A sparse chain about 0.4 to 4 eps apart, a few clumps, and a field 30 eps wide."""
    rng = np.random.default_rng(seed)
    chain = np.cumsum(rng.uniform(0.2, 3.0, size=(60, d)), axis=0) * (30.0 / 90.0)
    clumps = rng.uniform(0, 30, size=(4, d)).repeat(12, axis=0) + rng.uniform(0, 0.4, size=(48, d))
    p = np.concatenate([chain, clumps, rng.uniform(0, 30, size=(150, d))]) * eps
    return p[rng.permutation(len(p))].astype(np.float32)


@pytest.mark.parametrize("eps", [3e19, 1e-23])
@pytest.mark.parametrize("algo", ["densebox", "auto", "fdbscan"])
def test_three_points(dev, eps, algo):  # noqa: F811
    # 3.3 and 6.7 eps apart (2 and 4 eps), and all neighbours: eps^2 is infinite (0)
    x = np.array([0.0, 1e20, 2e20] if eps > 1 else [0.0, 2e-23, 4e-23], np.float32)
    pts = np.stack([x, np.zeros_like(x), np.zeros_like(x)], axis=1)
    ref = assert_exact(dev, pts, float(np.float32(eps)), 2, algo)
    assert ref[2] == 1


@pytest.mark.parametrize("eps", EPS)
@pytest.mark.parametrize("d", [2, 3])
def test_scene(dev, d, eps):  # noqa: F811
    e = float(np.float32(eps))
    pts = scene(d, eps, d)
    for min_pts in (2, 5):
        for algo in ("densebox", "fdbscan"):
            assert_exact(dev, pts, e, min_pts, algo)


@pytest.mark.parametrize("eps", [1e-23, 1e-20, 1.9e19, 3e19])
@pytest.mark.parametrize("d", [2, 3])
def test_cloud_of_a_batch(dev, d, eps):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    e = [float(np.float32(x)) for x in (0.25, eps, eps, 0.5)]
    mp = [3, 2, 5, 2]
    clouds = [scene(d, x, 3 * k + d) for k, x in enumerate(e)]
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    _say(f"[gpu] batch with eps {eps:g}, d={d}")
    for algo in ("densebox", "fdbscan"):
        lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), torch.from_numpy(off),
                                          torch.tensor(e, dtype=torch.float32), torch.tensor(mp, dtype=torch.int32),
                                          algo=algo)
        torch.cuda.synchronize()
        lab, core, k = lab.cpu().numpy(), core.cpu().numpy(), k.cpu().numpy()
        for c, p in enumerate(clouds):
            rl, rc, rk = oracle.dbscan(p, e[c], mp[c])
            s = slice(off[c], off[c + 1])
            assert k[c] == rk and np.array_equal(core[s], rc) and np.array_equal(lab[s], rl), (algo, c)
