"""Workloads that the pair counter is timed on, and their inputs.

The catalogues are the synthetic stand-ins of the benchmark: uniform points or
Neyman-Scott clusters (50 children per parent, Gaussian offsets of width sigma)
in a cube of side 420, with weights U(0.5, 1.5) where a statistic is weighted.
Bins are log-spaced.  Launch settings are left to the library (refine 0, the
default) except where a case names them.
"""
import numpy as np
import torch

from paper_1911_08275_amd import native

BOX = 420.0
CHILDREN = 50


def _case(**kw):
    c = dict(kind="xi", n=1000, n2=0, sigma=1.5, rmin=0.1, rmax=25.0, nbins=14, pimax=0.0, npi=1,
             precision="fp32", weighted=False, periodic=True, dtype="f64", refine="auto",
             unique=False, workspace=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a small sub-sample looked at interactively (launch and
        # synchronisation latency)
        _case(name="xi_2e3_uniform_f32", n=2_000, sigma=0.0, nbins=10),
        # the benchmark's first configuration: 10^4 uniform points, 20 bins, binary64
        _case(name="xi_1e4_uniform_f64", n=10_000, sigma=0.0, rmax=20.0, nbins=20,
              precision="fp64"),
        # a serving loop without allocation: 10^5 points, weighted mean separation
        _case(name="xi_noalloc_1e5_weighted", kind="xi_noalloc", n=100_003, weighted=True),
        # the headline: weighted xi of 10^6 clustered points, binary64
        _case(name="xi_1e6_weighted_f64", n=1_000_000, weighted=True, precision="fp64"),
        # the same catalogue's plain counts, binary32 filter and binary64 recheck
        _case(name="xi_1e6_f32", n=1_000_000),
        # small scales only (R_max 10): many light cells, binary64
        _case(name="xi_1e6_r10_f64", n=1_000_003, rmax=10.0, precision="fp64"),
        # large scales (R_max 80, the upper part of the R_max sweep)
        _case(name="xi_1e6_r80_f32", n=1_000_000, rmax=80.0),
        # projected correlation function: 14 r_p bins x 40 pi bins
        _case(name="wp_1e6_f32", kind="wp", n=1_000_000, pimax=40.0, npi=40),
        # the same statistic with the weighted mean r_p, binary64, an odd size
        _case(name="wp_250e3_weighted_f64", kind="wp", n=250_007, pimax=40.0, npi=40,
              weighted=True, precision="fp64"),
        # data x randoms of a survey: float32 inputs, not periodic, 10^6 x 10^7
        _case(name="cross_1e6_1e7_float32", kind="cross", n=1_000_000, n2=10_000_000,
              periodic=False, dtype="f32"),
        # weighted data x randoms in (r_p, pi), caller's workspace, not periodic
        _case(name="cross_wp_5e4_4e5_weighted", kind="cross_wp", n=50_021, n2=400_009, pimax=40.0,
              npi=20, rmax=30.0, nbins=12, weighted=True, periodic=False, workspace=True),
        # an MCMC step over a batch of mocks: xi and w_p of 16 catalogues of 2*10^5 to
        # 2*10^6 points, one plan (plan.execute + plan.results)
        _case(name="plan_16_mocks_f32", kind="plan", n=2_000_000, n2=200_000, nbins=14, pimax=40.0,
              npi=40, mocks=16),
    ]


def _sizes(c):
    """Catalogue sizes of a plan: spread evenly from n2 to n."""
    k = c["mocks"]
    return [int(round(c["n2"] + (c["n"] - c["n2"]) * i / max(1, k - 1))) for i in range(k)]


def _neighbours(c, n2):
    """Expected uniform points within reach of one point."""
    r = c["rmax"]
    v = np.pi * r * r * 2 * c["pimax"] if "wp" in c["kind"] else 4 / 3 * np.pi * r ** 3
    return n2 * v / BOX ** 3


def _pairs(c):
    """Expected in-range pairs that have to be evaluated."""
    if c["kind"] == "plan":
        return sum(_pairs(dict(c, kind="wp", n=n)) for n in _sizes(c))
    if c["kind"].startswith("cross"):
        return c["n"] * _neighbours(c, c["n2"])
    return 0.5 * c["n"] * (_neighbours(c, c["n"]) + (CHILDREN if c["sigma"] > 0 else 0))


def draw(rng):
    kind = rng.choice(["xi", "xi", "xi", "wp", "wp", "cross", "cross_wp", "xi_noalloc", "plan"])
    n = int(10 ** rng.uniform(3.2, 6.05)) | rng.randint(0, 1)
    c = _case(kind=kind, n=n, sigma=rng.choice([0.0, 0.7, 1.5, 3.0]),
              rmin=rng.choice([0.05, 0.1, 0.5]), rmax=round(10 ** rng.uniform(0.8, 1.6), 2),
              nbins=rng.randint(5, 30), precision=rng.choice(["fp32", "fp32", "fp64"]),
              weighted=rng.random() < 0.4, periodic=rng.random() < 0.7,
              dtype=rng.choice(["f64", "f64", "f32"]),
              refine=rng.choice(["auto", "auto", "2,2,2", "2,2,1", "1,1,1"]),
              unique=rng.random() < 0.2, workspace=rng.random() < 0.2)
    if kind == "xi_noalloc":
        c.update(n=min(n, 300_001), workspace=False)
    if "wp" in kind or kind == "plan":
        c.update(pimax=round(rng.uniform(1.0, 2.0) * c["rmax"], 1), npi=rng.choice([1, 10, 20, 40]))
    if kind.startswith("cross"):
        c.update(n=max(1000, n // 8), n2=n, unique=False)
    if kind == "plan":
        c.update(mocks=rng.randint(2, 9), weighted=False, periodic=True, workspace=False)
        c.update(n=max(2000, n // 2), n2=max(1000, n // 12))
    # no drawn case costs more than the largest listed one
    while _pairs(c) > 4e9:
        c.update(n=c["n"] // 2 + 1, n2=c["n2"] // 2 + 1 if c["n2"] else 0)
    return c


# ------------------------------------------------------------------ inputs

def _points(n, sigma, seed, dtype, weights):
    """(x, y, z, w): n points in [0, BOX)^3 on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if sigma > 0:
        parents = max(1, round(n / CHILDREN))
        centre = torch.rand((3, parents), generator=g, device="cuda", dtype=torch.float64) * BOX
        p = centre[:, torch.randint(0, parents, (n,), generator=g, device="cuda")]
        p += sigma * torch.randn((3, n), generator=g, device="cuda", dtype=torch.float64)
        p = torch.remainder(p, BOX)
        p[p >= BOX] = 0.0
    else:
        p = torch.rand((3, n), generator=g, device="cuda", dtype=torch.float64) * BOX
    w = None
    if weights:
        w = 0.5 + torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    if dtype == "f32":
        p = p.float()
        p = torch.clamp(p, max=float(np.nextafter(np.float32(BOX), np.float32(0))))
    return tuple(v.contiguous() for v in p) + (w,)


def _edges(c):
    return np.logspace(np.log10(c["rmin"]), np.log10(c["rmax"]), c["nbins"] + 1)


def _sets(c, seed):
    """The case's catalogues."""
    if c["kind"] == "plan":
        return [_points(n, c["sigma"], seed * 1000 + i, c["dtype"], False)
                for i, n in enumerate(_sizes(c))]
    a = [_points(c["n"], c["sigma"], seed * 1000, c["dtype"], c["weighted"])]
    if c["kind"].startswith("cross"):
        a.append(_points(c["n2"], 0.0, seed * 1000 + 1, c["dtype"], c["weighted"]))
    return a


def _options(c):
    o = dict(precision=c["precision"], periodic=c["periodic"],
             boxsize=BOX if c["periodic"] else 0.0, need_ravg=c["weighted"],
             count_mode="unique" if c["unique"] else "ordered")
    if c["refine"] != "auto":
        o["refine"] = tuple(int(v) for v in c["refine"].split(","))
    return o


def prepare(case, seed):
    c, edges, opt = case, _edges(case), _options(case)
    pts = [native.DevicePoints(*p) for p in _sets(c, seed)]
    s = dict(case=c, points=pts, edges=edges, options=opt)
    if c["kind"] == "plan":
        s["plan"] = native.Plan(pts, xi_edges=edges, wp_edges=edges, pimax=c["pimax"],
                                npibins=c["npi"], **opt)
    elif c["workspace"]:
        n2 = pts[1].n if len(pts) > 1 else 0
        size = native.workspace_size(c["kind"], pts[0].n, n2, edges, c["pimax"], c["npi"], **opt)
        opt["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    return s


def _outputs(r):
    d = {"npairs": r.npairs}
    if r.wsum is not None:
        d["wsum"], d["ravg"] = r.wsum, r.ravg
    return d


def run(state):
    c, pts, e, o = state["case"], state["points"], state["edges"], state["options"]
    if c["kind"] == "plan":
        state["plan"].execute()
        xi, wp = state["plan"].results()
        return {"xi": xi, "wp": wp}
    if c["kind"] == "xi":
        return _outputs(native.countpairs_xi(pts[0], e, **o))
    if c["kind"] == "xi_noalloc":
        return _outputs(native.countpairs_xi_noalloc(pts[0], e, **o))
    if c["kind"] == "wp":
        return _outputs(native.countpairs_wp(pts[0], e, c["pimax"], c["npi"], **o))
    if c["kind"] == "cross":
        return _outputs(native.countpairs_cross(pts[0], pts[1], e, **o))
    return _outputs(native.countpairs_cross_wp(pts[0], pts[1], e, c["pimax"], c["npi"], **o))


def work(case):
    """Bytes: every point read once, every output written once.  Operations: of
    each in-range pair (unique pairs of an auto-count) the squared separation
    (8) and, weighted, the weight product, the square root and two sums (5)."""
    c = case
    n = sum(_sizes(c)) if c["kind"] == "plan" else c["n"] + (c["n2"] if "cross" in c["kind"] else 0)
    per = 3 * (8 if c["dtype"] == "f64" else 4) + (8 if c["weighted"] else 0)
    out = 8 * c["nbins"] * (c["npi"] if "wp" in c["kind"] else 1) * (3 if c["weighted"] else 1)
    if c["kind"] == "plan":
        out = 8 * c["mocks"] * c["nbins"] * (1 + c["npi"])
    return {"bytes": n * per + out, "flops": _pairs(c) * (13 if c["weighted"] else 8)}


# ------------------------------------------------------------------- exact

def _minimum_image(d):
    d = torch.where(d > BOX / 2, d - BOX, d)
    return torch.where(d < -BOX / 2, d + BOX, d)


def exact(case, seed):
    """The counts and weighted sums from all pairs within reach along z, in
    binary64 by torch; None where that takes too long."""
    c = case
    if c["kind"] == "plan":
        return None
    wp, auto = "wp" in c["kind"], not c["kind"].startswith("cross")
    reach = c["pimax"] if wp else c["rmax"]
    n1, n2 = c["n"], c["n"] if auto else c["n2"]
    if n1 * n2 * min(1.0, (2 * reach + 5) / BOX) > 1.4e11:
        return None
    sets = [tuple(v.double() if v is not None else None for v in p) for p in _sets(c, seed)]
    a, b = sets[0], sets[-1]
    order = torch.argsort(b[2])
    bx, by, bz = (v[order] for v in b[:3])
    bw = b[3][order] if c["weighted"] else None
    if c["periodic"]:   # ghosts, so that a window in z is one range of the sorted points
        lo, hi = bz < reach + 1, bz > BOX - reach - 1
        idx = torch.cat([torch.nonzero(hi)[:, 0], torch.arange(n2, device="cuda"),
                         torch.nonzero(lo)[:, 0]])
        at = torch.cat([bz[hi] - BOX, bz, bz[lo] + BOX])
    else:
        idx, at = torch.arange(n2, device="cuda"), bz
    e = torch.from_numpy(_edges(c)).cuda()
    E = e * e
    nb, npi = c["nbins"], c["npi"] if wp else 1
    q = torch.arange(npi + 1, device="cuda", dtype=torch.float64) * (c["pimax"] / npi)
    q[npi] = c["pimax"]
    tot = [torch.zeros(nb * npi, dtype=torch.float64, device="cuda") for _ in range(3)]
    order1 = torch.argsort(a[2])
    rows = 1024 if n2 > 200_000 else 4096
    for i0 in range(0, n1, rows):
        i = order1[i0:i0 + rows]
        x, y, z = (v[i] for v in a[:3])
        j0 = int(torch.searchsorted(at, z[0] - reach - 1e-6))
        j1 = int(torch.searchsorted(at, z[-1] + reach + 1e-6))
        if c["periodic"] and (j1 - j0) > n2:
            j0, j1 = 0, 0   # the window is the whole box: every point once, as it is
            sel = torch.arange(n2, device="cuda")
        else:
            sel = idx[j0:j1]
        step = max(1, 80_000_000 // max(1, i.numel()))
        for k0 in range(0, sel.numel(), step):
            j = sel[k0:k0 + step]
            d = [p[j][None, :] - v[:, None] for p, v in ((bx, x), (by, y), (bz, z))]
            if c["periodic"]:
                d = [_minimum_image(v) for v in d]
            s = d[0] * d[0] + d[1] * d[1]
            if wp:
                keep = (s < E[-1]) & (d[2].abs() < c["pimax"])
            else:
                s = s + d[2] * d[2]
                keep = s < E[-1]
            keep &= s >= E[0]
            if auto:
                keep &= order[j][None, :] != i[:, None]
            r, col = torch.nonzero(keep, as_tuple=True)
            sk = s[r, col]
            bin_ = torch.bucketize(sk, E, right=True) - 1
            if wp:
                l = torch.bucketize(d[2][r, col].abs(), q, right=True) - 1
                bin_ = bin_ * npi + l
            # spread over 256 copies of the bins (one copy's sums would queue)
            many = bin_ * 256 + (r & 255)

            def sums(weights=None):
                v = torch.bincount(many, weights=weights, minlength=nb * npi * 256)
                return v.double().view(nb * npi, 256).sum(1)

            tot[0] += sums()
            if c["weighted"]:
                ww = a[3][i][r] * bw[j][col]
                tot[1] += sums(ww)
                tot[2] += sums(ww * torch.sqrt(sk))
    half = 0.5 if (auto and c["unique"]) else 1.0
    shape = (nb, npi) if wp else (nb,)
    n = (tot[0] * half).cpu().numpy().astype(np.uint64).reshape(shape)
    if not c["weighted"]:
        return {"npairs": n}
    w = tot[1].cpu().numpy()
    r = np.where(tot[0].cpu().numpy() > 0, tot[2].cpu().numpy() / np.where(w == 0, 1, w), 0.0)
    return {"npairs": n, "wsum": (w * half).reshape(shape), "ravg": r.reshape(shape)}
