"""Timed cases of the framework's public entry points.

Every case is one call (or, for the server, one burst of requests) as a
user's program makes it, on synthetic clouds of the kinds the repository's
benchmark and tests use, drawn on the GPU from a seed:

* ``surface``  d = 3 samples of a random ellipsoid or torus with N(0, 0.01^2)
  noise (two independent samples of one surface);
* ``mixture16`` 16 centres ~U[-10, 10]^d, sigma 1, B's centres moved by
  N(0, 0.5^2) (the small plain-method workload);
* ``clusters`` centres ~N(0, 4^2 I), sigma_j ~U[0.2, 1], A and B independent;
* ``tight``    many centres ~N(0, I), sigma 0.3 (the precision workload);
* ``mixed``    70% cluster points with Laplace(0, 0.5) noise around centres
  ~U[-50, 50]^d, 30% uniform in [-50, 50]^d;
* ``outlier``  standard Gaussian clouds, plus one point of A at
  0.5 n (1, ..., 1).

``listed`` gives the twelve timed cases, ``draw`` further ones over the same
ranges, ``prepare`` the inputs and handles a program holds before the call,
``run`` one pass, ``work`` the bytes and operations a pass cannot do without
and ``exact`` the outputs that have a value in 64 bits.
"""

import math
import weakref

import numpy as np
import torch

import paper_2307_03043_amd as ch

DEV = "cuda"
L1, L2 = ch.L1, ch.L2


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest request of the serving stream (1000..1500 points of a
        # d = 3 surface), called directly: latency and launches
        dict(name="est_l1_surface_1k_d3", kind="estimate", cloud="surface", metric=L1,
             n_a=1000, n_b=1371, d=3, eps=0.2, T=0, L=0, precision=0, reps=1),
        # the small plain-method workload with its own eps and T
        dict(name="est_l2_mixture_4k_d16", kind="estimate", cloud="mixture16", metric=L2,
             n_a=4096, n_b=4096, d=16, eps=0.2, T=512, L=0, precision=0, reps=1),
        # the small-scale protocol: symmetric estimate of two 20k-point
        # surfaces with the better CrudeNN of four LSH structures
        dict(name="est_sym_l1_surface_20k_d3", kind="estimate_sym", cloud="surface", metric=L1,
             n_a=20_000, n_b=19_001, d=3, eps=0.1, T=200, L=0, precision=0, reps=4),
        # the largest d = 3 requests of the serving stream, ragged sizes
        dict(name="est_l2_surface_200k_d3", kind="estimate", cloud="surface", metric=L2,
             n_a=199_999, n_b=150_011, d=3, eps=0.1, T=0, L=0, precision=0, reps=1),
        # the benchmark's default workload
        dict(name="est_l2_clusters_100k_d128", kind="estimate", cloud="clusters", metric=L2,
             n_a=100_000, n_b=100_000, d=128, eps=0.1, T=2000, L=20, precision=0, reps=1),
        # the l1 workload of the benchmark
        dict(name="est_l1_mixed_1m_d64", kind="estimate", cloud="mixed", metric=L1,
             n_a=1_000_000, n_b=1_000_000, d=64, eps=0.1, T=2000, L=24, precision=0, reps=1),
        # the benchmark's target point
        dict(name="est_l2_clusters_1m_d128", kind="estimate", cloud="clusters", metric=L2,
             n_a=1_000_000, n_b=1_000_000, d=128, eps=0.1, T=2000, L=24, precision=0, reps=1),
        # the precision workload: d = 256 with the BF16 exact pass
        dict(name="est_bf16_l2_tight_1m_d256", kind="estimate", cloud="tight", metric=L2,
             n_a=1_000_000, n_b=1_000_000, d=256, eps=0.1, T=2000, L=24, precision=1, reps=1),
        # brute force on the default workload: the exact answer itself
        dict(name="exact_l2_clusters_100k_d128", kind="exact", cloud="clusters", metric=L2,
             n_a=100_000, n_b=100_000, d=128, precision=0),
        # l1 brute force on the outlier scenario's clouds (d = 100, one odd row)
        dict(name="exact_l1_outlier_30k_d100", kind="exact", cloud="outlier", metric=L1,
             n_a=30_001, n_b=30_000, d=100, precision=0),
        # one-vs-many retrieval over a thousand d = 3 clouds, exact re-rank of 10
        dict(name="retrieve_l1_surface_1000", kind="retrieve", metric=L1, m=1000, n_min=1000,
             n_max=4000, eps=0.2, T=50, L=3, k=10),
        # a burst of 48 requests of the serving mix from pinned host memory
        dict(name="serve_mix_48", kind="serve", count=48, n_min=1000, n_max=200_000),
    ]


def _size(rng, lo, hi):
    """Log-uniform, odd as often as even."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["surface", "surface", "clusters", "clusters", "mixed", "tight",
                       "mixture16", "sym", "exact", "exact", "retrieve", "serve"])
    if kind == "retrieve":
        return dict(kind="retrieve", metric=rng.choice([L1, L1, L2]), m=_size(rng, 60, 1000),
                    n_min=1000, n_max=_size(rng, 1500, 4000), eps=0.2,
                    T=rng.choice([20, 50, 100]), L=rng.choice([3, 4]),
                    k=rng.choice([1, 5, 10, 30]))
    if kind == "serve":
        return dict(kind="serve", count=rng.randint(8, 48), n_min=1000,
                    n_max=_size(rng, 5000, 200_000))
    if kind == "sym":
        return dict(kind="estimate_sym", cloud="surface", metric=rng.choice([L1, L2]),
                    n_a=_size(rng, 1000, 100_000), n_b=_size(rng, 1000, 100_000), d=3,
                    eps=rng.choice([0.1, 0.2]), T=rng.choice([100, 200, 500]), L=0, precision=0,
                    reps=rng.choice([1, 4]))
    if kind == "exact":
        metric = rng.choice([L1, L2])
        cloud = rng.choice(["clusters", "mixed", "outlier", "surface"])
        d = 3 if cloud == "surface" else rng.choice([16, 50, 64, 100, 128])
        hi = 40_000 if metric == L2 or d == 3 else 30_000
        return dict(kind="exact", cloud=cloud, metric=metric, n_a=_size(rng, 2000, hi),
                    n_b=_size(rng, 2000, hi), d=d, precision=0)
    if kind == "surface":
        d, hi, metric = 3, 200_000, rng.choice([L1, L2])
    elif kind == "mixture16":
        d, hi, metric = 16, 20_000, L2
    elif kind == "mixed":
        d, hi, metric = rng.choice([32, 64, 100]), 600_000, L1
    elif kind == "tight":
        d, hi, metric = rng.choice([200, 256]), 300_000, L2
    else:
        d, hi, metric = rng.choice([64, 100, 128]), 600_000, rng.choice([L2, L2, L1])
    return dict(kind="estimate", cloud=kind, metric=metric, n_a=_size(rng, 1000, hi),
                n_b=_size(rng, 1000, hi), d=d, eps=rng.choice([0.1, 0.2]), T=0, L=0,
                precision=rng.choice([0, 1]) if kind == "tight" else 0, reps=1)


# ----------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _around(g, centres, sigma, n, laplace=False):
    """n points: a uniform choice of centre plus noise (row blocks, so that
    the temporaries of the largest clouds stay small)."""
    k, d = centres.shape
    out = torch.empty(n, d, device=DEV)
    for r in range(0, n, 1 << 18):
        m = min(n - r, 1 << 18)
        at = torch.randint(0, k, (m,), generator=g, device=DEV)
        if laplace:
            u = _uniform(g, m, d) - 0.5
            noise = -0.5 * torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999999))
        else:
            noise = _normal(g, m, d) * sigma[at][:, None]
        out[r:r + m] = centres[at] + noise
    return out


def _shapes(g, m):
    """m random surfaces: kind, (three axes | two radii), rotation."""
    kind = torch.randint(0, 2, (m,), generator=g, device=DEV)
    axes = 0.5 + 1.5 * _uniform(g, m, 3)
    radii = torch.stack([1.0 + _uniform(g, m), 0.2 + 0.3 * _uniform(g, m)], 1)
    q, r = torch.linalg.qr(_normal(g, m, 3, 3).cpu())
    rot = q * torch.sign(torch.diagonal(r, dim1=-2, dim2=-1))[:, None, :]
    return kind, axes, radii, rot.to(DEV)


def _sample(g, shapes, of):
    """One noisy point of surface of[i] for every i."""
    kind, axes, radii, rot = shapes
    n = of.numel()
    u = 2 * math.pi * _uniform(g, n)
    w = math.pi * _uniform(g, n)
    ell = torch.stack([w.sin() * u.cos(), w.sin() * u.sin(), w.cos()], 1) * axes[of]
    v = 2 * w
    ring = radii[of, 0] + radii[of, 1] * v.cos()
    tor = torch.stack([ring * u.cos(), ring * u.sin(), radii[of, 1] * v.sin()], 1)
    p = torch.where(kind[of][:, None] == 0, ell, tor)
    R = rot[of]
    p = (p[:, None, :] * R).sum(2)
    return (p + 0.01 * _normal(g, n, 3)).contiguous()


def _clouds(g, case):
    kind, n_a, n_b, d = case["cloud"], case["n_a"], case["n_b"], case["d"]
    if kind == "surface":
        s = _shapes(g, 1)
        return [_sample(g, s, torch.zeros(n, dtype=torch.int64, device=DEV)) for n in (n_a, n_b)]
    if kind == "mixture16":
        c = 20.0 * _uniform(g, 16, d) - 10.0
        one = torch.ones(16, device=DEV)
        return [_around(g, c, one, n_a), _around(g, c + 0.5 * _normal(g, 16, d), one, n_b)]
    if kind == "clusters":
        c = 4.0 * _normal(g, 1000, d)
        s = 0.2 + 0.8 * _uniform(g, 1000)
        return [_around(g, c, s, n) for n in (n_a, n_b)]
    if kind == "tight":
        c = _normal(g, 10_000, d)
        s = torch.full((10_000,), 0.3, device=DEV)
        return [_around(g, c, s, n) for n in (n_a, n_b)]
    if kind == "mixed":
        c = 100.0 * _uniform(g, 5000, d) - 50.0
        out = []
        for n in (n_a, n_b):
            x = _around(g, c, None, n, laplace=True)
            far = _uniform(g, n) < 0.3
            x[far] = 100.0 * _uniform(g, int(far.sum()), d) - 50.0
            out.append(x)
        return out
    a, b = _normal(g, n_a, d), _normal(g, n_b, d)
    a[-1] = 0.5 * n_a
    return [a, b]


class _Server:
    """A warmed server, closed with the state that holds it."""

    def __init__(self, arena, lanes):
        self.srv = ch.ChamferServer(arena, lanes)
        weakref.finalize(self, self.srv.close)
        for d in (3, 128):
            for metric in (L1, L2):
                self.srv.warm(d, metric)


def prepare(case, seed):
    g = _gen(seed)
    st = dict(case=case)
    if case["kind"] == "retrieve":
        m = case["m"]
        shapes = _shapes(g, m)
        sizes = torch.randint(case["n_min"], case["n_max"] + 1, (m,), generator=g, device=DEV)
        of = torch.repeat_interleave(torch.arange(m, device=DEV), sizes)
        st["Bs"] = _sample(g, shapes, of)
        st["sizes"] = sizes.tolist()
        src = seed % m  # the query is a resample of a member
        st["A"] = _sample(g, shapes, torch.full((st["sizes"][src],), src, device=DEV))
        st["seed"] = seed  # every query draws its own hash and samples
    elif case["kind"] == "serve":
        rng = np.random.default_rng(seed)
        lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
        reqs = []
        for i in range(case["count"]):
            surface = rng.uniform() < 0.8
            c = dict(cloud="surface" if surface else "clusters", d=3 if surface else 128,
                     n_a=int(round(math.exp(rng.uniform(lo, hi)))),
                     n_b=int(round(math.exp(rng.uniform(lo, hi)))))
            a, b = [x.cpu().pin_memory() for x in _clouds(g, c)]
            reqs.append((a, b, L2 if rng.uniform() < 0.7 else L1,
                         0.1 if rng.uniform() < 0.5 else 0.2, 0, seed + i))
        st["reqs"] = reqs
        st["server"] = _Server(2 << 30, 4)
    else:
        st["A"], st["B"] = _clouds(g, case)
        st["seed"] = 1  # one program-wide seed, as the benchmark's calls
    return st


# -------------------------------------------------------------- one pass

def run(st):
    c = st["case"]
    if c["kind"] == "estimate":
        return ch.chamfer_estimate(st["A"], st["B"], c["metric"], c["eps"], c["T"], st["seed"],
                                   n_scales=c["L"], precision=c["precision"], reps=c["reps"])
    if c["kind"] == "estimate_sym":
        return ch.chamfer_estimate_symmetric(st["A"], st["B"], c["metric"], c["eps"], c["T"],
                                             st["seed"], n_scales=c["L"],
                                             precision=c["precision"], reps=c["reps"])
    if c["kind"] == "exact":
        return ch.chamfer_exact(st["A"], st["B"], c["metric"], precision=c["precision"])
    if c["kind"] == "retrieve":
        return ch.chamfer_retrieve_packed(st["A"], st["Bs"], st["sizes"], c["metric"], c["eps"],
                                          c["T"], st["seed"], c["k"], n_scales=c["L"])
    srv = st["server"].srv
    ids = [srv.submit(*r) for r in st["reqs"]]
    got = {}
    while len(got) < len(ids):
        srv.progress()
        for r in srv.results():
            got[r["id"]] = r
    rows = [got[i] for i in ids]
    return dict(eta=np.array([r["eta"] for r in rows]), D=np.array([r["D"] for r in rows]),
                W=np.array([r["W"] for r in rows], np.int64),
                s=np.array([r["s"] for r in rows], np.int32),
                status=np.array([r["status"] for r in rows], np.int32))


# ------------------------------------------------- what a pass must do

def _default_T(n_a, eps):
    return math.ceil(math.ceil(math.log2(max(2, n_a))) / eps ** 2)


def _estimate_work(n_a, n_b, d, eps, T):
    """Both clouds read once, D_a, candidate and scale written; the exact
    distances of the T draws to all of B (a multiply-add, or a subtract and
    an add, per coordinate)."""
    T = T or _default_T(n_a, eps)
    return 4.0 * d * (n_a + n_b) + 12.0 * n_a + 12.0 * T, 2.0 * T * n_b * d


def work(case):
    if case["kind"] == "retrieve":
        n = (case["n_min"] + case["n_max"]) / 2
        b1, f1 = _estimate_work(n, n, 3, case["eps"], case["T"])
        exact = 2 * case["k"] * 2.0 * n * n * 3
        return dict(bytes=12.0 * n * (case["m"] + 1), flops=2 * case["m"] * f1 + exact)
    if case["kind"] == "serve":
        lo, hi = case["n_min"], case["n_max"]
        n = (hi - lo) / math.log(hi / lo)  # mean of a log-uniform size
        T = _default_T(n, 0.1) * 0.625     # eps 0.1 and 0.2 equally often
        d = 0.8 * 3 + 0.2 * 128
        return dict(bytes=case["count"] * 8.0 * n * d, flops=case["count"] * 2.0 * T * n * d)
    if case["kind"] == "exact":
        return dict(bytes=4.0 * case["d"] * (case["n_a"] + case["n_b"]) + 8.0 * case["n_a"],
                    flops=2.0 * case["n_a"] * case["n_b"] * case["d"])
    n_a, n_b, d = case["n_a"], case["n_b"], case["d"]
    b, f = _estimate_work(n_a, n_b, d, case["eps"], case["T"])
    if case["kind"] == "estimate_sym":
        f += _estimate_work(n_b, n_a, d, case["eps"], case["T"])[1]
    return dict(bytes=b, flops=f)


def exact(case, seed):
    """The brute force in float64: the sum and every row's minimum (the
    arg-min is a whole number).  The estimates depend on the hash and the
    draws of the method itself and have no other 64-bit value."""
    if case["kind"] != "exact":
        return None
    st = prepare(case, seed)
    A, B = st["A"].double(), st["B"].double()
    rows = []
    per = B.shape[0] * (B.shape[1] if case["metric"] == L1 else 1)
    step = max(1, min(4096, (1 << 28) // per))
    for r in range(0, A.shape[0], step):
        x = A[r:r + step]
        if case["metric"] == L1:
            rows.append((x[:, None, :] - B[None, :, :]).abs().sum(2).min(1).values)
        else:
            # nearest row by the expanded square, then its distance by differences
            at = (B.square().sum(1)[None, :] - 2.0 * (x @ B.t())).argmin(1)
            rows.append((x - B[at]).square().sum(1).sqrt())
    m = torch.cat(rows)
    return m.sum()[None], m, None
