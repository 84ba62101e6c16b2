"""Timed workloads of the clustering library, through its Python entry points.

Each case is one call (or one burst of served jobs) as a program makes it: points
in device memory, labels, core flags and cluster counts out. The inputs follow
the seeded generators of workloads/gen.py (Gaussian clumps over a uniform
background), drawn on the GPU; clump membership is drawn per point, so the input
order carries no locality, as in the shuffled originals. Where `n` differs from a
generator's own size, the domain's side and the number of clumps grow with it, so
the local density (and with it the work per point) stays the same.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2103_05162_amd as fdb

# Point sets: dimension, the size the generator is quoted at, its clumps (number
# and width), the share of points in them, eps and minPts.
SETS = {
    # GPS-like blobs in the plane (the 16,384-point set of the tests and the benchmark)
    "blobs2d": dict(dim=2, n=16384, clumps=8, sigma=(0.01, 0.01), share=0.7, eps=0.01, min_pts=5),
    # friends-of-friends halos: clumps of unequal mass and width, minPts 2
    "fof3d": dict(dim=3, n=2097152, clumps=2000, sigma=(0.002, 0.02), share=0.8, eps=0.005, min_pts=2, unequal=True),
    # very dense clumps over a thin background (the headline set)
    "dense3d": dict(dim=3, n=8388608, clumps=500, sigma=(5e-4, 5e-4), share=0.8, eps=0.002, min_pts=10),
    # no clumps at all, about four neighbours expected per point: no dense cells
    "uniform3d": dict(dim=3, n=2097152, clumps=0, sigma=(0.0, 0.0), share=0.0,
                      eps=(4.0 / (2097152 * 4.0 / 3.0 * math.pi)) ** (1.0 / 3.0), min_pts=5),
}

SERVE_BUDGET = 8 << 30  # the server's default device budget


def listed():
    return [
        # the smallest call that is worth making: a frame's detections or a tile of
        # a map, where the latency of the launches and of the returned K is all there is
        dict(name="densebox_2d_1k", kind="single", set="blobs2d", algo="densebox", n=1021),
        # the 16,384-point 2D set, both algorithms (FDbscan is the entry point's default)
        dict(name="densebox_2d_16k", kind="single", set="blobs2d", algo="densebox", n=16384),
        dict(name="fdbscan_2d_16k", kind="single", set="blobs2d", algo="fdbscan", n=16384),
        # one request of ordinary size (the served trace's mean), a few clumps in a unit cube
        dict(name="densebox_3d_370k", kind="single", set="mixture3d", algo="densebox", n=370003, eps=0.0125,
             min_pts=5),
        # a large planar set of ragged size
        dict(name="densebox_2d_1m", kind="single", set="blobs2d", algo="densebox", n=1000003),
        # sparse data without dense cells, the automatic choice
        dict(name="auto_3d_uniform_2m", kind="single", set="uniform3d", algo="auto", n=2097152),
        # friends-of-friends halo finding, both algorithms
        dict(name="densebox_3d_fof_2m", kind="single", set="fof3d", algo="densebox", n=2097152),
        dict(name="fdbscan_3d_fof_2m", kind="single", set="fof3d", algo="fdbscan", n=2097152),
        # the headline set, both algorithms
        dict(name="densebox_3d_dense_8m", kind="single", set="dense3d", algo="densebox", n=8388608),
        dict(name="fdbscan_3d_dense_8m", kind="single", set="dense3d", algo="fdbscan", n=8388608),
        # many uneven clouds in one call (about 65M points)
        dict(name="batched_3d_4096", kind="batched", dim=3, algo="densebox", clouds=4096, lo=1024, hi=65536, min_pts=5),
        # a burst of requests to the continuous-batching server, 2D and 3D mixed
        dict(name="served_24_jobs", kind="served", algo="densebox", jobs=24, lo=10240, hi=2097152),
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    what = rng.choice(["single"] * 7 + ["batched"] * 2 + ["served"])
    if what == "batched":
        return dict(kind="batched", dim=rng.choice([2, 3]), algo=rng.choice(["densebox", "densebox", "fdbscan"]),
                    clouds=_log_uniform(rng, 16, 1024), lo=rng.choice([64, 1024]), hi=rng.choice([8192, 32768]),
                    min_pts=rng.choice([2, 5, 10]))
    if what == "served":
        return dict(kind="served", algo="densebox", jobs=rng.randint(4, 24), lo=rng.choice([1000, 10240]),
                    hi=rng.choice([200000, 2097152]))
    name = rng.choice(["blobs2d", "mixture2d", "mixture3d", "fof3d", "dense3d", "uniform3d"])
    algo = rng.choice(["densebox", "densebox", "fdbscan", "auto"])
    # FDbscan tests every pair within eps: a few wide-eps clumps of many points are DenseBox's case
    top = 100000 if name.startswith("mixture") and algo == "fdbscan" else 2097152 if algo == "fdbscan" else 8388608
    if name == "uniform3d":
        top = min(top, 4194304)
    c = dict(kind="single", set=name, algo=algo, n=_log_uniform(rng, 1000, top) | 1,
             border=rng.choice(["canonical", "canonical", "canonical", "none"]))
    if name.startswith("mixture"):
        c.update(eps=round(rng.uniform(0.005, 0.02), 5), min_pts=rng.choice([2, 5, 10]))
    else:
        base = SETS[name]
        # sets of few neighbours per point are all noise at a large minPts
        few = name in ("fof3d", "uniform3d")
        c.update(eps=base["eps"] * round(rng.uniform(0.8, 1.1), 3), min_pts=rng.choice([2, 5] if few else [2, 5, 10, 30]))
    return c


# ---- inputs ------------------------------------------------------------------------


def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64)


def _clumps(gen, n, dim, side, centers, sigma, weight, share):
    """n points, a share of them in clumps drawn by weight, the rest uniform in [0, side]^dim."""
    pts = _rand(gen, n, dim) * side
    if centers is not None:
        cum = torch.cumsum(weight, 0)
        which = torch.searchsorted(cum, _rand(gen, n) * cum[-1]).clamp_(max=centers.shape[0] - 1)
        noise = torch.randn(n, dim, generator=gen, device="cuda", dtype=torch.float64)
        inside = (_rand(gen, n) < share).unsqueeze(1)
        pts = torch.where(inside, centers[which] + sigma[which].unsqueeze(1) * noise, pts)
    return pts.to(torch.float32)


def _mixture(gen, n, dim):
    """A few clumps of log-uniform width in the unit cube with 10% noise: one cloud of a batch or a trace."""
    k = int(torch.randint(1, 21, (1,), generator=gen, device="cuda"))
    sigma = torch.exp(_rand(gen, k) * math.log(10.0) + math.log(0.002))
    return _clumps(gen, n, dim, 1.0, _rand(gen, k, dim), sigma, torch.ones(k, device="cuda", dtype=torch.float64), 0.9)


def _set_points(case, gen):
    n = case["n"]
    if case["set"].startswith("mixture"):
        return _mixture(gen, n, int(case["set"][-2]))
    s = SETS[case["set"]]
    d, scale = s["dim"], n / s["n"]
    side = scale ** (1.0 / d)
    if not s["clumps"]:
        return _clumps(gen, n, d, side, None, None, None, 0.0)
    k = max(1, round(s["clumps"] * scale))
    lo, hi = s["sigma"]
    med = math.sqrt(lo * hi)
    sigma = torch.full((k,), med, device="cuda", dtype=torch.float64)
    weight = torch.ones(k, device="cuda", dtype=torch.float64)
    if s.get("unequal"):
        sd = math.log(hi / med) / 2.0
        normal = torch.randn(2, k, generator=gen, device="cuda", dtype=torch.float64)
        sigma = (sigma * torch.exp(normal[0] * sd)).clamp_(lo, hi)
        weight = torch.exp(normal[1])
    return _clumps(gen, n, d, side, _rand(gen, k, d) * side, sigma, weight, s["share"])


def _sizes(case):
    """Sizes of a batch's clouds or a burst's jobs: log-uniform, fixed by the case."""
    rng = np.random.default_rng([4, case.get("clouds", 0), case.get("jobs", 0), case["lo"], case["hi"]])
    count = case["clouds"] if case["kind"] == "batched" else case["jobs"]
    return np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=count)).astype(np.int64)


def _batch(case, gen):
    """Every cloud a mixture of its own, drawn for all clouds at once."""
    dim, sizes = case["dim"], torch.from_numpy(_sizes(case)).cuda()
    b, n = sizes.numel(), int(sizes.sum())
    k = torch.randint(1, 21, (b,), generator=gen, device="cuda")
    centers = _rand(gen, b * 20, dim)
    sigma = torch.exp(_rand(gen, b * 20) * math.log(10.0) + math.log(0.002))
    cloud = torch.repeat_interleave(torch.arange(b, device="cuda"), sizes)
    which = cloud * 20 + (_rand(gen, n) * k[cloud]).long()
    inside = (_rand(gen, n) < 0.9).unsqueeze(1)
    points = torch.empty(n, dim, device="cuda", dtype=torch.float32)
    for a in range(dim):  # an axis at a time: the largest batch has 65M points
        clump = centers[which, a] + sigma[which] * torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
        points[:, a] = torch.where(inside[:, 0], clump, _rand(gen, n)).to(torch.float32)
    offsets = torch.zeros(b + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(sizes, 0)
    eps = (0.005 + 0.015 * _rand(gen, b)).to(torch.float32)
    return points, offsets, eps, torch.full((b,), case["min_pts"], dtype=torch.int32, device="cuda")


def _jobs(case, gen):
    jobs = []
    for k, n in enumerate(_sizes(case)):
        dim = 2 + k % 2
        eps = float(np.float32(0.005 + 0.015 * float(_rand(gen, 1))))
        jobs.append(dict(points=_mixture(gen, int(n), dim), n=int(n), dim=dim, eps=eps, min_pts=(2, 5, 10)[k % 3],
                         labels=torch.empty(int(n), dtype=torch.int32, device="cuda"),
                         core=torch.empty(int(n), dtype=torch.uint8, device="cuda")))
    return jobs


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = dict(case=case)
    if case["kind"] == "single":
        base = SETS.get(case["set"], {})
        state.update(points=_set_points(case, gen), eps=float(np.float32(case.get("eps", base.get("eps")))),
                     min_pts=case.get("min_pts", base.get("min_pts")))
    elif case["kind"] == "batched":
        state["batch"] = _batch(case, gen)
    else:
        state["jobs"] = _jobs(case, gen)
        state["server"] = fdb.Server(budget_bytes=SERVE_BUDGET, algo=case["algo"])
        torch.cuda.synchronize()  # a job's points are ready before it is submitted
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "single":
        labels, core, k = fdb.dbscan(state["points"], state["eps"], state["min_pts"], algo=case["algo"],
                                     border=case.get("border", "canonical"))
        return dict(labels=labels, core=core, k=k)
    if case["kind"] == "batched":
        points, offsets, eps, min_pts = state["batch"]
        labels, core, k = fdb.dbscan_batched(points, offsets, eps, min_pts, algo=case["algo"])
        return dict(labels=labels, core=core, k=k)
    server, jobs = state["server"], state["jobs"]
    tickets = [server.submit_raw(j["points"].data_ptr(), j["n"], j["dim"], j["eps"], j["min_pts"],
                                 j["labels"].data_ptr(), j["core"].data_ptr()) for j in jobs]
    k = [server.wait(t)["num_clusters"] for t in tickets]
    return dict(labels=[j["labels"] for j in jobs], core=[j["core"] for j in jobs], k=np.asarray(k, dtype=np.int32))


def work(case):
    """Points in, labels and core flags out; and the distance tests that decide a
    core point: at least minPts - 1 other points within eps have to be seen."""
    if case["kind"] == "single":
        s = SETS.get(case["set"], {})
        dims, n, m = [s.get("dim") or int(case["set"][-2])], [case["n"]], case.get("min_pts", s.get("min_pts"))
    else:
        n = [int(x) for x in _sizes(case)]
        dims = [case["dim"]] * len(n) if case["kind"] == "batched" else [2 + k % 2 for k in range(len(n))]
        m = case.get("min_pts", 5)
    return dict(bytes=sum(c * (4 * d + 5) for c, d in zip(n, dims)),
                flops=sum(c * (m - 1) * 3 * d for c, d in zip(n, dims)))


def exact(case, seed):
    """Labels, core flags and counts are whole numbers: nothing is rounded on the way out."""
    return None
