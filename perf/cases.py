"""Workloads of the library over the range it is used on: pair counts of angular and 3-D catalogs from a thousand
points to a few million, in both precisions, with and without tile pruning, split by jackknife region, batched, and
served as jobs whose catalogs arrive from the host.

Catalogs are seeded stand-ins for survey data: blobs on a uniform background for the data, uniform randoms."""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1204_6630_amd as tp
from paper_1204_6630_amd import serving

PATCH = (0.0, 30.0, 0.0, 30.0)      # RA and Dec ranges in degrees
OCTANT = (0.0, 90.0, 0.0, 90.0)
BOX = 1000.0                        # side of the 3-D box


def listed():
    return [
        # the smallest request a serving loop meets: one synchronous DD count of a thousand objects
        {"name": "dd_1e3", "path": "count", "sky": "patch", "nd": 1000, "nr": 0, "bins": 20, "lo": 0.01, "hi": 10.0,
         "fp64": False, "prune": False},
        # w(theta) of a small field: DD, DR, RR and the estimator, 1e4 objects, sizes off every tile
        {"name": "w_patch_1e4", "path": "step", "sky": "patch", "nd": 10007, "nr": 9973, "bins": 20, "lo": 0.01,
         "hi": 10.0, "fp64": False, "prune": False},
        # w(theta) of an octant with 1e5 objects and as many randoms
        {"name": "w_octant_1e5", "path": "step", "sky": "octant", "nd": 100000, "nr": 100000, "bins": 30,
         "lo": 0.001, "hi": 20.0, "fp64": False, "prune": False},
        # the survey-sized w(theta): 1e6 objects, 2e6 randoms, 4.5e12 pairs
        {"name": "w_octant_1e6x2e6", "path": "step", "sky": "octant", "nd": 1000000, "nr": 2000000, "bins": 40,
         "lo": 0.0005, "hi": 30.0, "fp64": False, "prune": False},
        # edges out to 120 deg, no pair beyond the last edge
        {"name": "w_octant_to120deg", "path": "step", "sky": "octant", "nd": 200003, "nr": 400009, "bins": 40,
         "lo": 0.0005, "hi": 120.0, "fp64": False, "prune": False},
        # many narrow bins (two-byte tables), a medium field
        {"name": "w_octant_200bins", "path": "step", "sky": "octant", "nd": 100003, "nr": 200003, "bins": 200,
         "lo": 0.01, "hi": 30.0, "fp64": False, "prune": False},
        # the plain FP64 path
        {"name": "w_octant_fp64", "path": "step", "sky": "octant", "nd": 150001, "nr": 300007, "bins": 40,
         "lo": 0.0005, "hi": 30.0, "fp64": True, "prune": False},
        # exact tile pruning, as a survey pipeline that wants the counts soonest sets it
        {"name": "w_octant_pruned", "path": "step", "sky": "octant", "nd": 500000, "nr": 1000000, "bins": 40,
         "lo": 0.0005, "hi": 30.0, "fp64": False, "prune": True},
        # the spatial xi(r) in a box
        {"name": "xi_box_5e5x1e6", "path": "step", "sky": "box", "nd": 500000, "nr": 1000000, "bins": 30, "lo": 0.5,
         "hi": 150.0, "fp64": False, "prune": False},
        # w(theta) with delete-one jackknife errors over an 8 x 8 grid of regions
        {"name": "w_jackknife_64", "path": "regions", "sky": "octant", "nd": 100000, "nr": 200000, "bins": 30,
         "lo": 0.05, "hi": 20.0, "fp64": False, "prune": False, "grid": 8},
        # many fields of uneven size against one random catalog in one launch, replayed as a graph
        {"name": "batch_24", "path": "batch", "sky": "octant", "nd": 50000, "nr": 200000, "bins": 30, "lo": 0.001,
         "hi": 20.0, "fp64": False, "prune": False, "jobs": 24},
        # a burst of serving jobs: catalogs uploaded from the host, DD or DR against resident randoms, released
        {"name": "serve_12", "path": "serve", "sky": "octant", "nd": 100000, "nr": 300000, "bins": 30, "lo": 0.001,
         "hi": 20.0, "fp64": False, "prune": False, "jobs": 12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["count", "step", "step", "step", "step", "regions", "batch", "serve"])
    sky = rng.choice(["patch", "octant", "octant", "octant", "box"])
    c = {"path": path, "sky": sky, "fp64": rng.random() < 0.2, "prune": rng.random() < 0.2}
    if path == "count":
        c.update(nd=_log_int(rng, 1000, 300000), nr=0)
    elif path == "step":
        top = 200000 if c["fp64"] else 700000
        c.update(nd=_log_int(rng, 2000, top), nr=_log_int(rng, 2000, 2 * top))
    else:
        c.update(nd=_log_int(rng, 5000, 100000), nr=_log_int(rng, 20000, 300000))
    c["bins"] = rng.choice([1, 8, 20, 30, 40, 64, 120, 200, 256])
    if sky == "box":
        c.update(lo=rng.uniform(0.2, 2.0), hi=rng.uniform(60.0, 300.0))
    elif sky == "patch":
        c.update(lo=rng.uniform(0.005, 0.1), hi=rng.uniform(3.0, 30.0))
    else:
        c.update(lo=10.0 ** rng.uniform(-3.3, -1.0), hi=rng.uniform(5.0, 120.0))
    if path == "regions":
        c["grid"] = rng.choice([2, 3, 5, 8])
    elif path in ("batch", "serve"):
        c.update(sky="octant", jobs=rng.randint(4, 24), lo=10.0 ** rng.uniform(-3.0, -1.0), hi=rng.uniform(5.0, 60.0))
    return c


# ---------------------------------------------------------------------------
# inputs

def _uniform(n, fp, g):
    ra = g.uniform(fp[0], fp[1], n)
    dec = np.degrees(np.arcsin(g.uniform(math.sin(math.radians(fp[2])), math.sin(math.radians(fp[3])), n)))
    return ra, dec


def _clustered(n, fp, sigma, g):
    """70 % of the points in blobs of 50 around uniform centres, the rest uniform; blob points that leave the
    footprint are drawn uniformly."""
    k = int(0.7 * n)
    cra, cdec = _uniform(max(1, k // 50), fp, g)
    at = g.integers(0, cra.size, k)
    a, d, s = np.radians(cra[at]), np.radians(cdec[at]), math.radians(sigma)
    xi, eta = g.normal(0.0, s, k), g.normal(0.0, s, k)
    ca, sa, cd, sd = np.cos(a), np.sin(a), np.cos(d), np.sin(d)
    x, y, z = cd * ca - xi * sa - eta * sd * ca, cd * sa + xi * ca - eta * sd * sa, sd + eta * cd
    r = np.sqrt(x * x + y * y + z * z)
    bra, bdec = np.degrees(np.arctan2(y, x)) % 360.0, np.degrees(np.arcsin(np.clip(z / r, -1.0, 1.0)))
    ura, udec = _uniform(n, fp, g)
    ok = (bra >= fp[0]) & (bra < fp[1]) & (bdec >= fp[2]) & (bdec < fp[3])
    ura[:k][ok], udec[:k][ok] = bra[ok], bdec[ok]
    perm = g.permutation(n)
    return ura[perm], udec[perm]


def _points(case, n, g, clustered):
    """(ra, dec) in degrees, or (x, y, z) in the box."""
    if case["sky"] == "box":
        p = g.uniform(0.0, BOX, (3, n))
        if clustered:
            k = int(0.7 * n)
            c = g.uniform(0.0, BOX, (3, max(1, k // 35)))
            q = c[:, g.integers(0, c.shape[1], k)] + g.normal(0.0, 2.0, (3, k))
            ok = np.all((q >= 0.0) & (q < BOX), axis=0)
            p[:, :k][:, ok] = q[:, ok]
            p = p[:, g.permutation(n)]
        return tuple(np.ascontiguousarray(v) for v in p)
    fp = PATCH if case["sky"] == "patch" else OCTANT
    if case["path"] in ("batch", "serve") and clustered:
        a0, d0 = g.uniform(0.0, 70.0), g.uniform(0.0, 70.0)
        fp = (a0, a0 + 20.0, d0, d0 + 20.0)
    return _clustered(n, fp, 0.3, g) if clustered else _uniform(n, fp, g)


def _regions(case, pts):
    """Labels of a grid over the footprint (3-D: over x and y)."""
    k = case["grid"]
    fp = (0.0, BOX, 0.0, BOX) if case["sky"] == "box" else PATCH if case["sky"] == "patch" else OCTANT
    i = np.clip(((pts[0] - fp[0]) / (fp[1] - fp[0]) * k).astype(np.int64), 0, k - 1)
    j = np.clip(((pts[1] - fp[2]) / (fp[3] - fp[2]) * k).astype(np.int64), 0, k - 1)
    return (j * k + i).astype(np.int32)


def _edges(case):
    a, b, n = math.log10(case["lo"]), math.log10(case["hi"]), case["bins"]
    e = np.array([10.0 ** (a + k * (b - a) / n) for k in range(n + 1)])
    e[0], e[-1] = case["lo"], case["hi"]
    return e


def _job_sizes(case):
    """Catalog sizes of a batch or a burst: spread over a factor of 50 below nd (the same for every seed)."""
    g = np.random.default_rng(case["jobs"])
    return [max(2, int(case["nd"] / 50.0 ** u)) for u in g.uniform(0.0, 1.0, case["jobs"])]


def _inputs(case, seed):
    g = np.random.default_rng(seed)
    if case["path"] in ("batch", "serve"):
        data = [_points(case, n, g, True) for n in _job_sizes(case)]
    else:
        data = [_points(case, case["nd"], g, True)]
    randoms = _points(case, case["nr"], g, False) if case["nr"] else None
    return data, randoms


def _upload(ctx, case, pts, labels=None):
    box = case["sky"] == "box"
    if labels is not None:
        k = case["grid"] ** 2
        return ctx.upload_catalog_3d_regions(*pts, labels, k) if box else ctx.upload_catalog_regions(*pts, labels, k)
    return ctx.upload_catalog_3d(*pts) if box else ctx.upload_catalog(*pts)


# ---------------------------------------------------------------------------
# one pass

def prepare(case, seed):
    data, randoms = _inputs(case, seed)
    ctx = tp.Context(0)
    if case["prune"]:
        ctx.set_tuning(prune=1)
    st = {"case": case, "ctx": ctx, "edges": _edges(case), "prec": tp.FP64 if case["fp64"] else tp.FP32_CHORD}
    path = case["path"]
    st["sizes"] = [p[0].size for p in data]
    if path == "regions":
        ld, lr = _regions(case, data[0]), _regions(case, randoms)
        st["cd"], st["cr"] = _upload(ctx, case, data[0], ld), _upload(ctx, case, randoms, lr)
        st["nd_reg"], st["nr_reg"] = ctx.catalog_regions(st["cd"]), ctx.catalog_regions(st["cr"])
    elif path == "serve":
        st["cr"] = _upload(ctx, case, randoms)
        st["data"] = data
    else:
        st["cats"] = [_upload(ctx, case, p) for p in data]
        st["cr"] = _upload(ctx, case, randoms) if randoms is not None else -1
    if path == "step":
        st["out"] = torch.zeros((3, case["bins"] + 2), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
    if path == "batch":
        jobs = []
        for c in st["cats"]:
            jobs += [(tp.DD, c, -1), (tp.DR, c, st["cr"])]
        st["jobs"] = jobs + [(tp.RR, st["cr"], -1)]
    return st


def run(st):
    case, ctx, e, prec = st["case"], st["ctx"], st["edges"], st["prec"]
    path = case["path"]
    if path == "count":
        return ctx.count(tp.DD, st["cats"][0], e, precision=prec)
    if path == "step":
        out, cd, cr = st["out"], st["cats"][0], st["cr"]
        ctx.count_async(tp.DD, cd, e, out[0].data_ptr(), precision=prec)
        ctx.count_async(tp.DR, cd, e, out[1].data_ptr(), cat_b=cr, precision=prec)
        ctx.count_async(tp.RR, cr, e, out[2].data_ptr(), precision=prec)
        ctx.synchronize()
        h = out.cpu().numpy()
        w = tp.landy_szalay(h[0].view(np.uint64), h[1].view(np.uint64), h[2].view(np.uint64), case["nd"], case["nr"])
        return {"counts": h, "w": w}
    if path == "regions":
        cd, cr = st["cd"], st["cr"]
        dd, dd_t = ctx.count_regions(tp.DD, cd, e, precision=prec)
        dr, dr_t = ctx.count_regions(tp.DR, cd, e, cat_b=cr, precision=prec)
        rr, rr_t = ctx.count_regions(tp.RR, cr, e, precision=prec)
        samples, mean, cov = tp.jackknife(dd, dd_t, dr, dr_t, rr, rr_t, case["nd"], st["nd_reg"], case["nr"],
                                          st["nr_reg"])
        return {"totals": np.stack([dd, dr, rr]), "touch": np.stack([dd_t, dr_t, rr_t]), "samples": samples,
                "mean": mean, "cov": cov}
    if path == "batch":
        return ctx.count_batch(st["jobs"], e, precision=prec, graph=True)
    jobs = [serving.Job(id=k, kind="DD" if k % 2 else "DR", arrival=0.0, ra=p[0], dec=p[1], n=p[0].size)
            for k, p in enumerate(st["data"])]
    srv = serving.Server(serving.LibraryBackend(ctx, e, prec), [st["cr"]], case["nr"])
    rep = srv.run(jobs)
    return np.stack([rep.results[k] for k in range(len(jobs))])


def _pairs(case):
    nd, nr = case["nd"], case["nr"]
    if case["path"] == "count":
        return nd * (nd - 1) // 2
    if case["path"] in ("step", "regions"):
        return nd * (nd - 1) // 2 + nd * nr + nr * (nr - 1) // 2
    sizes = _job_sizes(case)
    if case["path"] == "batch":
        return sum(n * (n - 1) // 2 + n * nr for n in sizes) + nr * (nr - 1) // 2
    return sum(n * (n - 1) // 2 if k % 2 else n * nr for k, n in enumerate(sizes))


def work(case):
    """Each point's coordinates read once and each histogram written once; five operations form a pair's dot
    product (eight its squared distance) and one bins it."""
    n = case["nr"] + (sum(_job_sizes(case)) if case["path"] in ("batch", "serve") else case["nd"])
    slots = (case["bins"] + 2) * 8 * (3 if case["path"] in ("step", "regions") else case.get("jobs", 1))
    if case["path"] == "regions":
        slots *= 1 + case["grid"] ** 2
    return {"bytes": n * (24 if case["fp64"] else 12) + slots,
            "flops": _pairs(case) * (9 if case["sky"] == "box" else 6)}


# ---------------------------------------------------------------------------
# the same in plain FP64

MOST_PAIRS = 8e10       # about 20 seconds on the GPU


def _vectors(case, pts, dev):
    if case["sky"] == "box":
        return [torch.from_numpy(v).to(dev) for v in pts]
    a, d = np.radians(pts[0]), np.radians(pts[1])
    return [torch.from_numpy(v).to(dev) for v in (np.cos(d) * np.cos(a), np.cos(d) * np.sin(a), np.sin(d))]


def _separations(case, a, b):
    if case["sky"] == "box":
        dx, dy, dz = (u[:, None] - v[None, :] for u, v in zip(a, b))
        return torch.sqrt((dx * dx + dy * dy) + dz * dz)
    x, y, z = (u[:, None] * v[None, :] for u, v in zip(a, b))
    return torch.acos(torch.clamp((x + y) + z, -1.0, 1.0))


def _count(case, a, b, edges, la, lb, k):
    """Slot counts of all ordered pairs (i in a, j in b) by region pair: (k, k, nslots); all labels 0 without
    regions.  Slot = the number of edges at or below the separation."""
    dev = a[0].device
    n = b[0].numel()
    past = torch.zeros((k, len(edges) + 1, k), dtype=torch.int64, device=dev)
    for r in range(k):
        rows = torch.nonzero(la == r).flatten()
        col = torch.zeros((len(edges) + 1, n), dtype=torch.int64, device=dev)
        col[0] = rows.numel()
        step = max(1, (1 << 27) // max(1, n))
        for s in range(0, rows.numel(), step):
            i = rows[s:s + step]
            t = _separations(case, [v[i] for v in a], b)
            for q, e in enumerate(edges):
                col[q + 1] += (t >= e).sum(0)
        past[r].index_add_(1, lb, col)
    past = past.permute(0, 2, 1)
    return torch.cat([past[..., :-1] - past[..., 1:], past[..., -1:]], -1).cpu().numpy()


def _histograms(case, a, b, edges, la, lb, k):
    """Unordered pairs i < j when b is None, all pairs otherwise: (total, touch by region)."""
    if b is not None:
        h = _count(case, a, b, edges, la, lb, k)
        touch = h.sum(1) + h.sum(0) - h[np.arange(k), np.arange(k)]
        return h.sum((0, 1)), touch
    h = _count(case, a, a, edges, la, la, k)
    if case["sky"] == "box":
        self_sep = torch.zeros_like(a[0])
    else:
        self_sep = torch.acos(torch.clamp((a[0] * a[0] + a[1] * a[1]) + a[2] * a[2], -1.0, 1.0))
    slot = (self_sep[:, None] >= torch.tensor(edges, device=a[0].device)[None, :]).sum(1).cpu().numpy()
    np.subtract.at(h, (la.cpu().numpy(), la.cpu().numpy(), slot), 1)
    diag = h[np.arange(k), np.arange(k)] // 2
    total = h.sum((0, 1)) // 2
    touch = h.sum(1) - diag         # a pair across regions is in h twice, one inside a region too
    return total, touch


def _estimate(dd, dr, rr, nd, nr):
    rr_n = np.where(rr[1:-1] > 0, rr[1:-1] / (nr * (nr - 1.0) / 2.0), np.nan)
    return (dd[1:-1] / (nd * (nd - 1.0) / 2.0) - 2.0 * (dr[1:-1] / (nd * float(nr))) + rr_n) / rr_n


def exact(case, seed):
    cuda = torch.cuda.is_available()
    if _pairs(case) * (case["bins"] + 9) / 40 > (MOST_PAIRS if cuda else 4e8):
        return None
    dev = torch.device("cuda" if cuda else "cpu")
    data, randoms = _inputs(case, seed)
    edges = _edges(case)
    if case["sky"] != "box":
        edges = edges * (math.pi / 180.0)
    edges = [float(e) for e in edges]
    path, k = case["path"], case["grid"] ** 2 if case["path"] == "regions" else 1
    vec = lambda p: _vectors(case, p, dev)                                                  # noqa: E731
    lab = lambda p: torch.from_numpy(_regions(case, p).astype(np.int64)).to(dev) if k > 1 else \
        torch.zeros(p[0].size, dtype=torch.int64, device=dev)                               # noqa: E731
    if path in ("count", "batch", "serve"):
        r = vec(randoms) if randoms is not None else None
        got = []
        for q, p in enumerate(data):
            a = vec(p)
            if path != "serve" or q % 2:
                got.append(_histograms(case, a, None, edges, lab(p), None, 1)[0])
            if path == "batch" or (path == "serve" and not q % 2):
                got.append(_histograms(case, a, r, edges, lab(p), lab(randoms), 1)[0])
        if path == "batch":
            got.append(_histograms(case, r, None, edges, lab(randoms), None, 1)[0])
        return got[0] if path == "count" else np.stack(got)
    d, r, ld, lr = vec(data[0]), vec(randoms), lab(data[0]), lab(randoms)
    tot, touch = zip(_histograms(case, d, None, edges, ld, None, k), _histograms(case, d, r, edges, ld, lr, k),
                     _histograms(case, r, None, edges, lr, None, k))
    nd, nr = case["nd"], case["nr"]
    with np.errstate(divide="ignore", invalid="ignore"):
        if path == "step":
            return {"counts": np.stack(tot), "w": _estimate(*tot, nd, nr)}
        cd, cr = np.bincount(ld.cpu().numpy(), minlength=k), np.bincount(lr.cpu().numpy(), minlength=k)
        samples = np.stack([_estimate(*(t - u[q] for t, u in zip(tot, touch)), nd - int(cd[q]), nr - int(cr[q]))
                            for q in range(k)])
        mean = samples.mean(0)
        dev_ = samples - mean
        cov = (k - 1.0) / k * (dev_.T @ dev_)
    return {"totals": np.stack(tot), "touch": np.stack(touch), "samples": samples, "mean": mean, "cov": cov}
