"""Kernels that only large inputs reach, on scenes whose labels are known without a search.
DenseBox above 524,288 points, where the walks through the grid and through the hierarchy are
kernels of their own (`far`: one point so far out that the hierarchy serves), with many dense
cells (a lane each), fewer and larger ones (a wavefront each) and none. And batches whose
number of points lies at the edges of the sort's tiles and of its one launch, in narrow grids,
so that pairs of key digits are the same for every point."""
import numpy as np
import pytest

from tests.test_gpu_parity import _say, dev, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def groups(n, d, size, chain, spacing, seed, width=0.25):
    """Groups of `size` points on a lattice, in shuffled order: in a box `width` wide, or
    (chain) in a row 0.8 apart. Returns the points, each point's group, and its place in the group."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n)
    g, place = perm // size, perm % size
    side = int(np.ceil((-(-n // size)) ** (1.0 / d)))
    at = np.stack([g // side**k % side for k in range(d)], axis=1) * float(spacing)
    off = rng.uniform(0.0, width, size=(n, d))
    if chain:
        off[:, 0] = 0.8 * place
    return (at + off).astype(np.float32), g, place


def ranked(g, core, member):
    """Cluster ids in the order of each group's smallest core index; -1 outside groups."""
    idx = np.flatnonzero(core)
    _, first = np.unique(g[idx], return_index=True)
    ids = np.full(g.max() + 1, -1, np.int64)
    ids[g[np.sort(idx[first])]] = np.arange(first.size)
    return np.where(member, ids[g], -1)


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("kind", ["lanes", "wavefronts", "chains"])
@pytest.mark.parametrize("border", ["canonical", "first", "none"])
def test_large_densebox(dev, far, d, kind, border):  # noqa: F811
    n = 524288 + 40
    size = {"lanes": 4, "wavefronts": 20, "chains": 5}[kind]
    # (narrow groups: nearly all of them in one cell each, more than 65,536 of them)
    pts, g, place = groups(n, d, size, kind == "chains", 10, d, width=0.01 if kind == "lanes" else 0.25)
    count = np.bincount(g)[g]
    if kind == "chains":  # minPts 3: a row's inner points are core, its ends are border points
        core, member = (place > 0) & (place < count - 1), count > 2
    else:
        core = member = count >= 3
    if far:
        pts = np.concatenate([pts, np.full((1, d), 1.0e7, np.float32)])
        g, core, member = np.append(g, g.max() + 1), np.append(core, False), np.append(member, False)
    _say(f"[gpu] {kind} far={far} d={d} {border}")
    lab, got, k = run_gpu(dev, pts, 1.0, 3, "densebox", border=border)
    want = ranked(g, core, member & core if border == "none" else member)
    assert k == want.max() + 1 and np.array_equal(got.astype(bool), core)
    if border == "first":
        pairs = np.unique(np.stack([lab, want], axis=1), axis=0)
        assert len(pairs) == len(np.unique(lab)) == len(np.unique(want))
        assert np.array_equal(lab < 0, want < 0)
    else:
        assert np.array_equal(lab, want)


@pytest.mark.parametrize("algo", ["fdbscan", "densebox"])
@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("n", [32768, 32769, 131072, 131073, 262144, 262145])
@pytest.mark.parametrize("num", [3, 70])
def test_batch_sort_edges(dev, algo, d, n, num):  # noqa: F811
    import torch
    import paper_2103_05162_amd as fdb
    rng = np.random.default_rng(n + num)
    cut = np.sort(rng.choice(np.arange(1, n), num - 1, replace=False))
    off = np.concatenate([[0], cut, [n]]).astype(np.int64)
    clouds = [groups(int(b - a), d, 4, False, 10, int(a)) for a, b in zip(off[:-1], off[1:])]
    _say(f"[gpu] batch sort {algo} d={d} n={n} clouds={num}")
    lab, core, k = fdb.dbscan_batched(torch.from_numpy(np.concatenate([c[0] for c in clouds])).to(dev),
                                      torch.from_numpy(off), torch.ones(num), torch.full((num,), 2, dtype=torch.int32),
                                      algo=algo)
    torch.cuda.synchronize()
    lab, core, k = lab.cpu().numpy(), core.cpu().numpy(), k.cpu().numpy()
    for c, (_, g, _) in enumerate(clouds):
        s = slice(off[c], off[c + 1])
        want_core = np.bincount(g)[g] >= 2
        want = ranked(g, want_core, want_core) if want_core.any() else np.full(g.size, -1)
        assert k[c] == want.max() + 1 and np.array_equal(core[s], want_core) and np.array_equal(lab[s], want), c
