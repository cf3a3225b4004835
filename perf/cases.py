"""Workloads of the library as a program uses it: whole passes from a star
field to its critical curves, caustics and source-plane maps, and the map and
lens-map calls on their own, over the range of field sizes, phase grids,
precisions and star sums that the library takes.

A case is a dict of plain values with a "kind":
  field    set_lenses, find_critical_curves with the caustics, the crossing map
           and the distance map of one circular field
  rect     the same for a rectangular field
  batched  set_lenses_batched and find_critical_curves over many fields
  maps     crossing map, distance map, moving-source distances and their
           histograms from caustics already in hand
  lensmap  map_caustics at arbitrary points of the lens plane
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2506_02121_amd import fields
from paper_2506_02121_amd.mlcc import Context, Grid

MEAN_SALPETER = 0.1674   # mean of dN/dm ~ m^-2.35 on [0.08, 1]


def _half(n, masses, kappa_star, part):
    """Half-width of a source-plane window: `part` of the field's radius."""
    mean = 1.0 if masses == "equal" else MEAN_SALPETER
    return round(part * math.sqrt(n * mean / kappa_star), 3)


def listed():
    return [
        # the smallest field in use: launches, copies and waits decide
        dict(name="field_tiny", kind="field", n=10, masses="equal", kappa_star=0.3, kappa_s=0.0,
             gamma=0.3, m_steps=1000, precision="fp64", star_sums="direct", half=8.0, npix=256),
        # a small field at an odd size in the mixed form, as a parameter scan runs them
        dict(name="field_small_mixed", kind="field", n=137, masses="salpeter", kappa_star=0.4,
             kappa_s=0.1, gamma=0.25, m_steps=2000, precision="mixed", star_sums="direct",
             half=5.0, npix=500),
        # the 1,000-star field of the benchmark, whole
        dict(name="field_n1k", kind="field", n=1000, masses="salpeter", kappa_star=0.4,
             kappa_s=0.2, gamma=0.45, m_steps=10000, precision="fp64", star_sums="direct",
             half=10.0, npix=1024),
        # the benchmark's headline settings in the default precision, on a field and a phase grid
        # that keep a pass near a second (the headline's 10,000 stars and 20,000 steps take five)
        dict(name="field_n6k", kind="field", n=6000, masses="equal", kappa_star=0.5,
             kappa_s=0.0, gamma=0.3, m_steps=10000, precision="fp64", star_sums="direct",
             half=16.0, npix=2048),
        # a large field with unequal masses in the mixed form
        dict(name="field_n4k_mixed", kind="field", n=4099, masses="salpeter", kappa_star=0.6,
             kappa_s=0.0, gamma=0.4, m_steps=6000, precision="mixed", star_sums="direct",
             half=8.0, npix=1024),
        # FP64 with multipole star sums
        dict(name="field_n3k_fmm", kind="field", n=3000, masses="salpeter", kappa_star=0.4,
             kappa_s=0.0, gamma=0.3, m_steps=6000, precision="fp64", star_sums="fmm",
             half=10.0, npix=1024),
        # the headline field whole, in its fastest form
        dict(name="field_n10k_mixed_fmm", kind="field", n=10000, masses="equal", kappa_star=0.5,
             kappa_s=0.0, gamma=0.3, m_steps=20000, precision="mixed", star_sums="fmm",
             half=20.0, npix=2048),
        # a rectangular field over the headline's source window
        dict(name="rect_n437", kind="rect", n=437, masses="equal", kappa_star=0.5, kappa_s=0.0,
             gamma=0.3, t=87, m_steps=10000, precision="fp64", half=20.0, npix=1024),
        # many realisations in one call, sizes spread as in the benchmark's batch
        dict(name="batched_mixed", kind="batched", n_fields=40, n_lo=50, n_hi=2500, m_steps=2000,
             precision="mixed", star_sums="direct"),
        # the same use with multipole sums and many small fields
        dict(name="batched_small_fmm", kind="batched", n_fields=96, n_lo=50, n_hi=600,
             m_steps=1000, precision="mixed", star_sums="fmm"),
        # the maps alone, at the headline's resolution, from a dense caustic network
        dict(name="maps_2048", kind="maps", rows=2001, loops=6000, nx=2048, ny=2048, angles=4,
             bins=400, size=0.02),
        # the lens map at points of the user's choice
        dict(name="lensmap_1m", kind="lensmap", n=1000, masses="salpeter", kappa_star=0.4,
             kappa_s=0.2, gamma=0.45, count=1000003),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["field", "field", "field", "rect", "batched", "maps", "lensmap"])
    masses = rng.choice(["equal", "salpeter"])
    ks = round(rng.uniform(0.2, 0.7), 3)
    smooth = round(rng.choice([0.0, rng.uniform(0.0, 0.2)]), 3)
    gamma = round(rng.uniform(0.05, 0.55), 3)
    if kind in ("field", "rect"):
        precision, star_sums = rng.choice([("fp64", "direct"), ("mixed", "direct"),
                                           ("fp64_r32", "direct"), ("fp64", "fmm"),
                                           ("mixed", "fmm")])
        n = _log(rng, 10, 6000 if kind == "field" else 600)
        # phase steps: fewer for larger fields, as their direct sums cost N^2 a row
        m = min(_log(rng, 800, 12000), int(1.0e11 / (n * n)))
        m -= m % 8
        npix = _log(rng, 100, 2048)
        c = dict(kind=kind, n=n, masses=masses, kappa_star=ks, kappa_s=smooth, gamma=gamma,
                 m_steps=m, precision=precision, star_sums=star_sums,
                 half=_half(n, masses, ks, 0.4), npix=npix)
        if kind == "rect":   # solved in the FP64 precisions; t from its truncation rule
            c.update(precision="fp64", t=rng.choice([9, 21, 43, 87]))
            c.pop("star_sums")
        return c
    if kind == "batched":
        hi = _log(rng, 200, 2500)
        nf = rng.randint(8, max(9, min(120, int(60000 / hi))))
        return dict(kind="batched", n_fields=nf, n_lo=rng.randint(10, 100), n_hi=hi,
                    m_steps=8 * rng.randint(100, 250), precision=rng.choice(["mixed", "fp64"]),
                    star_sums=rng.choice(["direct", "fmm"]))
    if kind == "maps":
        return dict(kind="maps", rows=_log(rng, 200, 2001), loops=_log(rng, 20, 6000),
                    nx=_log(rng, 200, 2048), ny=_log(rng, 200, 2048), angles=rng.randint(1, 4),
                    bins=rng.randint(20, 800), size=round(rng.uniform(0.01, 0.05), 4))
    n = _log(rng, 10, 4000)
    return dict(kind="lensmap", n=n, masses=masses, kappa_star=ks, kappa_s=smooth, gamma=gamma,
                count=min(_log(rng, 10000, 4000000), int(1.0e9 / n)))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _field(case, rng):
    if case["kind"] == "rect":
        aspect = (1.0 + case["gamma"]) / (1.0 - case["gamma"])
        t = case["t"]
        # the nearest degree clear of the leading coefficient's zeros
        arg = math.atan(aspect)
        while not 0.12 * math.pi <= math.fmod((t - 1) * arg, math.pi) <= 0.88 * math.pi:
            t += 2
        return fields.make_rect_field(rng, case["n"], case["kappa_star"], case["kappa_s"],
                                      case["gamma"], aspect, t, case["masses"])
    return fields.make_field(rng, case["n"], case["kappa_star"], case["kappa_s"], case["gamma"],
                             case["masses"])


def _loops(case, rng):
    """Clockwise astroid caustics, each split over two columns that continue
    each other (as the chains of a two-image caustic do): vertex planes
    (rows, 2 loops) and chain_next, over a window of unit height per 2048
    pixels."""
    rows, nl = case["rows"], case["loops"]
    w, h = case["nx"] / 2048.0, case["ny"] / 2048.0
    cx = _dev((rng.random(nl) - 0.5) * 1.2 * w)
    cy = _dev((rng.random(nl) - 0.5) * 1.2 * h)
    s = _dev(case["size"] * np.exp(0.5 * rng.standard_normal(nl)))
    tilt = _dev(2.0 * np.pi * rng.random(nl))
    re = torch.empty((rows, 2 * nl), dtype=torch.float64, device="cuda")
    im = torch.empty_like(re)
    for part in (0, 1):
        p = -(torch.arange(rows, dtype=torch.float64, device="cuda") / (rows - 1) + part) * math.pi
        x, y = torch.cos(p)[:, None] ** 3 * s, torch.sin(p)[:, None] ** 3 * s
        re[:, part::2] = cx + x * torch.cos(tilt) - y * torch.sin(tilt)
        im[:, part::2] = cy + x * torch.sin(tilt) + y * torch.cos(tilt)
    nxt = torch.arange(2 * nl, dtype=torch.int32, device="cuda") ^ 1
    return re, im, nxt, w, h


def prepare(case, seed):
    rng = np.random.default_rng([int(seed), 17, case.get("n", case.get("n_fields", 1))])
    st = dict(case=dict(case), ctx=Context(0))
    kind = case["kind"]
    if kind in ("field", "rect"):
        f = _field(case, rng)
        st.update(x=_dev(f.x), y=_dev(f.y), m=_dev(f.m), sheet=f.sheet,
                  grid=Grid(0.0, 0.0, case["half"], case["half"], case["npix"], case["npix"]))
    elif kind == "batched":
        # the sizes belong to the case, what fills them to the seed
        sizes = np.random.default_rng([case["n_fields"], case["n_lo"], case["n_hi"]])
        fs = []
        for _ in range(case["n_fields"]):
            n = int(round(math.exp(sizes.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
            ks, g = float(rng.uniform(0.1, 0.8)), float(rng.uniform(0.0, 0.6))
            fs.append(fields.make_field(rng, n, ks, 0.0, g, "salpeter"))
        off = np.concatenate([[0], np.cumsum([f.n for f in fs])])
        st.update(x=_dev(np.concatenate([f.x for f in fs])),
                  y=_dev(np.concatenate([f.y for f in fs])),
                  m=_dev(np.concatenate([f.m for f in fs])), off=[int(v) for v in off],
                  kappa_s=[f.kappa_s for f in fs], gamma=[f.gamma for f in fs])
    elif kind == "maps":
        re, im, nxt, w, h = _loops(case, rng)
        st.update(re=re, im=im, next=nxt,
                  grid=Grid(0.0, 0.0, 0.5 * w, 0.5 * h, case["nx"], case["ny"]),
                  angles=[float(a) for a in rng.uniform(0.0, 2.0 * math.pi, case["angles"])],
                  d_max=0.2 * max(w, h))
    else:
        f = _field(case, rng)
        r = 1.2 * f.radius
        st.update(zr=_dev(rng.uniform(-r, r, case["count"])),
                  zi=_dev(rng.uniform(-r, r, case["count"])), f=f)
        # the lenses stay loaded while points are mapped
        st["ctx"].set_lenses(_dev(f.x), _dev(f.y), _dev(f.m), f.kappa_s, f.gamma)
    return st


def run(st):
    c, ctx = st["case"], st["ctx"]
    kind = c["kind"]
    if kind in ("field", "rect"):
        if kind == "rect":
            ctx.set_lenses_rect(st["x"], st["y"], st["m"], c["kappa_s"], c["gamma"], *st["sheet"])
        else:
            ctx.set_lenses(st["x"], st["y"], st["m"], c["kappa_s"], c["gamma"])
        rr, ri, cr, ci, nxt, _, _ = ctx.find_critical_curves(
            c["m_steps"], precision=c["precision"], star_sums=c.get("star_sums", "direct"),
            caustics=True)
        ncc = ctx.caustic_crossings(cr, ci, nxt, st["grid"])
        dist, border = ctx.caustic_distances(st["grid"], ncc)
        return dict(roots_re=rr, roots_im=ri, caustics_re=cr, caustics_im=ci, chain_next=nxt,
                    ncc=ncc, dist=dist, border=border)
    if kind == "batched":
        ctx.set_lenses_batched(st["off"], st["x"], st["y"], st["m"], st["kappa_s"], st["gamma"])
        rr, ri, cr, ci, nxt, _, _ = ctx.find_critical_curves(
            c["m_steps"], precision=c["precision"], star_sums=c["star_sums"], caustics=True)
        return dict(roots_re=rr, roots_im=ri, caustics_re=cr, caustics_im=ci, chain_next=nxt)
    if kind == "maps":
        ncc = ctx.caustic_crossings(st["re"], st["im"], st["next"], st["grid"])
        dist, border = ctx.caustic_distances(st["grid"], ncc)
        out = dict(ncc=ncc, dist=dist, border=border)
        for i, a in enumerate(st["angles"]):
            d, b = ctx.caustic_distances_directional(st["grid"], ncc, a)
            out[f"dist_{i}"], out[f"border_{i}"] = d, b
            out[f"hist_{i}"] = ctx.distance_histogram(d, b, c["bins"], st["d_max"])
        out["hist_ncc"] = ctx.distance_histogram(dist, border, c["bins"], st["d_max"], ncc=ncc,
                                                 n_classes=4)
        return out
    return ctx.map_caustics(st["zr"], st["zi"])


def _mean_n(case):
    """Mean of N and of N^2 over a batch's log-uniform sizes."""
    lo, hi = case["n_lo"], case["n_hi"]
    if hi <= lo:
        return float(lo), float(lo) ** 2
    d = math.log(hi / lo)
    return (hi - lo) / d, (hi * hi - lo * lo) / (2.0 * d)


def work(case):
    """One update per root and row: 29 operations per star term of a direct
    sum; with multipole sums 27 near stars and a series of 48 terms.  The
    root-root sums can be had from expansions of groups of roots, so they are
    not counted.  Bytes: every root and caustic written once, every pixel of
    each map written once, the map's input read once."""
    kind = case["kind"]
    px = 13.0   # an int32 count, a float64 distance, a mark

    def star(n1, n2, fmm):   # operations for all roots of a row: sum over fields
        return 2.0 * (n1 * (29.0 * 27.0 + 26.0 * 48.0) if fmm else 29.0 * n2)

    if kind in ("field", "rect"):
        n, m = float(case["n"]), case["m_steps"]
        n_r = 2.0 * n + (case["t"] - 1 if kind == "rect" else 0)
        s = star(n, n * n, case.get("star_sums") == "fmm") * n_r / (2.0 * n)
        return {"bytes": (m + 1) * n_r * 48.0 + 24.0 * n + 17.0 * case["npix"] ** 2,
                "flops": m * s}
    if kind == "batched":
        n1, n2 = _mean_n(case)
        m = case["m_steps"]
        return {"bytes": case["n_fields"] * ((m + 1) * 2.0 * n1 * 32.0 + 24.0 * n1),
                "flops": case["n_fields"] * m * star(n1, n2, case["star_sums"] == "fmm")}
    if kind == "maps":
        p = float(case["nx"]) * case["ny"]
        return {"bytes": case["rows"] * case["loops"] * 32.0 + p * (px + 4.0) +
                case["angles"] * p * (px + 9.0) + 13.0 * p, "flops": 0.0}
    return {"bytes": 32.0 * case["count"] + 24.0 * case["n"],
            "flops": 12.0 * case["n"] * case["count"]}


def exact(case, seed):
    """The lens map in 64 bits from plain tensor operations.  The roots have
    no closed form, and their columns are numbered by the cold start."""
    if case["kind"] != "lensmap":
        return None
    st = prepare(case, seed)
    f, zr, zi = st["f"], st["zr"], st["zi"]
    sx, sy, sm = _dev(f.x), _dev(f.y), _dev(f.m)
    wr, wi = torch.empty_like(zr), torch.empty_like(zi)
    step = max(1, (1 << 26) // f.n)
    for a in range(0, zr.numel(), step):
        x, y = zr[a:a + step, None], zi[a:a + step, None]
        dx, dy = x - sx, y - sy
        v = sm / (dx * dx + dy * dy)
        wr[a:a + step] = (1.0 - f.kappa_s + f.gamma) * x[:, 0] - (v * dx).sum(1)
        wi[a:a + step] = (1.0 - f.kappa_s - f.gamma) * y[:, 0] - (v * dy).sum(1)
    return wr, wi
