"""Performance cases of the pair-counting library: what a program that
measures correlation functions calls, from one catalog of a few thousand
points to the full light cone and the angular cap.

A case is a dict of plain values. ``prepare`` draws its catalogs on the GPU
(float64 positions, shuffled order, shapes of ``catalogs``: periodic and open
boxes with Gaussian blobs, the redshift-shaped light cone, angular caps) and
makes the binning; ``run`` is one pass from positions to counts through the
public entry points (grid build included, since every new catalog pays it).
"""
import math

import numpy as np
import torch

import paper_1210_1833_amd as cute

C_OVER_H0 = 2997.92458  # Mpc/h

PREC = {"fp32_edge": cute.PREC_FP32_EDGE, "fp64": cute.PREC_FP64}


def listed():
    return [
        # the smallest call: a kept grid of a small sub-box counted again and
        # again by a loop that must not allocate (noalloc entry point)
        {"name": "noalloc_small", "path": "noalloc", "n": 2003, "box": 464.0, "r_max": 100.0, "n1": 20},
        # one small mock: monopole of a periodic box of 2e4 points, xi against
        # the uniform expectation
        {"name": "box_mono_2e4", "path": "box", "n": 20000, "blob_frac": 0.0, "box": 1000.0, "r_max": 150.0,
         "n1": 30, "log": False, "prec": "fp32_edge"},
        # the benchmark's step: r-mu DD of 1e6 strongly clustered points
        {"name": "rmu_dd_1e6", "path": "rmu_dd", "n": 1000000, "box": 2000.0, "r_max": 200.0, "n1": 40, "n2": 50,
         "prec": "fp32_edge"},
        # the same count with the all-FP64 classifier (a user's cross-check)
        {"name": "rmu_dd_fp64_4e5", "path": "rmu_dd", "n": 400000, "box": 1473.6, "r_max": 200.0, "n1": 40,
         "n2": 50, "prec": "fp64"},
        # a whole correlation function: DD, DR and RR, Landy-Szalay, multipoles
        {"name": "rmu_xi_25e4", "path": "rmu_xi", "n": 250007, "n_rand": 500029, "box": 1260.0, "r_max": 200.0,
         "n1": 40, "n2": 50},
        # the light cone at full size: sigma-pi DD, 75 x 75 bins
        {"name": "sigmapi_dd_3e6", "path": "sigmapi", "n": 3000000, "n_rand": 0, "ra": 60.0, "dec": 30.0,
         "r_max": 150.0, "n1": 75, "n2": 75},
        # a survey subset, r-mu against the pair midpoint: data-random counts
        {"name": "rmu_mid_dr_12e4", "path": "rmu_mid", "n": 120011, "n_rand": 240007, "ra": 18.0, "dec": 18.0,
         "r_max": 120.0, "n1": 24, "n2": 20},
        # angular correlation of a clustered cap, four decades of theta
        {"name": "theta_dd_2e6", "path": "theta", "n": 2000000, "half_angle": 40.75, "theta_min": 0.001,
         "theta_max": 10.0, "n1": 30, "prec": "fp32_edge"},
        # pixelised w(theta) of a survey subset: both maps and the weighted DR
        {"name": "wpix_dr_3e5", "path": "wpix", "n": 300000, "n_rand": 300000, "n_cth": 2048, "n_phi": 4028,
         "theta_max": 30.0, "n1": 256},
        # radial correlation of the same subset (one degree aperture)
        {"name": "radial_dr_3e5", "path": "radial", "n": 300000, "n_rand": 300000, "aperture": 1.0, "dz": 0.1,
         "n1": 100},
        # a batch of mocks for a covariance: monopole and r-mu of each
        {"name": "batch_12_mocks", "path": "batch", "mocks": 12, "n_lo": 20000, "n_hi": 100000, "box": 1000.0},
        # jackknife of one catalog: 100 column regions, r-mu
        {"name": "jackknife_25e4", "path": "jackknife", "n": 250000, "box": 1000.0, "side": 10, "r_max": 150.0,
         "n1": 30, "n2": 50},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | (rng.random() < 0.5)


def draw(rng):
    """One more case: a path, then sizes log-uniform over its range at the
    listed densities, and its options."""
    path = rng.choice(["noalloc", "box", "rmu_dd", "rmu_dd", "rmu_xi", "sigmapi", "rmu_mid", "theta", "wpix", "radial",
                       "batch", "jackknife"])
    c = {"path": path}
    if path == "noalloc":
        n = _size(rng, 1000, 20000)
        c.update(n=n, box=round(1000.0 * (n / 20000.0) ** (1 / 3.0), 1), r_max=rng.choice([40.0, 60.0, 100.0]),
                 n1=rng.choice([10, 20, 27]))
        c["r_max"] = min(c["r_max"], round(0.3 * c["box"], 1))
    elif path == "box":
        n = _size(rng, 20000, 1000000)
        c.update(n=n, blob_frac=rng.choice([0.0, 0.5]), box=1000.0, r_max=rng.choice([30.0, 100.0, 150.0]),
                 n1=rng.choice([15, 30, 100, 255]), log=rng.random() < 0.4, prec="fp32_edge")
    elif path == "rmu_dd":
        n = _size(rng, 20000, 1000000)
        prec = rng.choice(["fp32_edge", "fp32_edge", "fp64"])
        c.update(n=n, box=round(2000.0 * (n / 1e6) ** (1 / 3.0), 1), r_max=rng.choice([60.0, 120.0, 150.0, 200.0]),
                 n1=rng.choice([20, 40, 61]), n2=rng.choice([10, 50, 100]), prec=prec)
        c["r_max"] = min(c["r_max"], round(0.3 * c["box"], 1))
    elif path == "rmu_xi":
        n = _size(rng, 10000, 500000)
        c.update(n=n, n_rand=2 * n + rng.randrange(100), box=round(2000.0 * (n / 1e6) ** (1 / 3.0), 1),
                 r_max=rng.choice([100.0, 150.0, 200.0]), n1=rng.choice([20, 40]), n2=rng.choice([20, 50]))
        c["r_max"] = min(c["r_max"], round(0.3 * c["box"], 1))
    elif path == "sigmapi":
        f = math.exp(rng.uniform(math.log(0.02), 0.0))
        nr = rng.choice([0, 1])
        n = _size(rng, 3000000 * f * 0.9, 3000000 * f) if not nr else _size(rng, 400000 * f * 0.9, 400000 * f)
        r = rng.choice([40.0, 80.0, 150.0])
        c.update(n=n, n_rand=2 * n * nr, ra=round(60.0 * math.sqrt(f), 2), dec=round(30.0 * math.sqrt(f), 2),
                 r_max=r, n1=rng.choice([20, 40, 75]), n2=rng.choice([20, 75]))
    elif path == "rmu_mid":
        n = _size(rng, 15000, 300000)
        c.update(n=n, n_rand=2 * n, ra=18.0, dec=18.0, r_max=rng.choice([50.0, 100.0, 120.0]),
                 n1=rng.choice([10, 24, 50]), n2=rng.choice([10, 20, 100]))
    elif path == "theta":
        f = math.exp(rng.uniform(math.log(0.01), 0.0))
        n = _size(rng, 2000000 * f * 0.9, 2000000 * f)
        tmax = rng.choice([1.0, 5.0, 10.0])
        c.update(n=n, half_angle=round(max(40.75 * math.sqrt(f), tmax), 2), theta_min=rng.choice([0.0, 0.001, 0.01]),
                 theta_max=tmax, n1=rng.choice([20, 30, 64]), prec="fp32_edge")
    elif path == "wpix":
        n = _size(rng, 30000, 1000000)
        k = rng.choice([512, 1024, 2048])
        c.update(n=n, n_rand=n, n_cth=k, n_phi=2 * k - 68, theta_max=rng.choice([10.0, 20.0, 30.0]),
                 n1=rng.choice([64, 256]))
    elif path == "radial":
        n = _size(rng, 20000, 600000)
        c.update(n=n, n_rand=rng.choice([0, n]), aperture=rng.choice([0.2, 0.5, 1.0]), dz=0.1, n1=rng.choice([50, 100]))
    elif path == "batch":
        c.update(mocks=rng.randrange(4, 25), n_lo=_size(rng, 15000, 30000), n_hi=_size(rng, 40000, 150000), box=1000.0)
    else:
        n = _size(rng, 30000, 500000)
        c.update(n=n, box=1000.0, side=rng.choice([4, 7, 10]), r_max=rng.choice([80.0, 150.0]), n1=rng.choice([20, 30]),
                 n2=rng.choice([20, 50]))
    return c


# ---------------------------------------------------------------------------
# catalogs on the GPU (the shapes of catalogs/, drawn with torch)
# ---------------------------------------------------------------------------
def _gen(seed, role):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + role)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _columns(g, p):
    """(x, y, z) columns of the points in a random order."""
    p = p[torch.randperm(p.shape[0], generator=g, device="cuda")]
    return [p[:, k].contiguous() for k in range(3)]


def _box(g, n, box, blob_frac, wrap, per=100, sigma=5.0):
    """n points in a box: a share of them in Gaussian blobs of 100 points,
    the rest uniform; folded back into the box when it is periodic."""
    nb = int(n * blob_frac) // per
    u = _rand(g, n - nb * per, 3) * box
    b = (_rand(g, nb, 1, 3) * box + sigma * _normal(g, nb, per, 3)).reshape(-1, 3)
    p = torch.cat([u, b])
    if wrap:
        p = torch.remainder(p, box)
        p = torch.where(p >= box, torch.zeros_like(p), p)
    return _columns(g, p)


def _chi_table():
    z = np.arange(0.0, 3.0, 1e-3)
    e = 1.0 / np.sqrt(0.3 * (1.0 + z) ** 3 + 0.7)
    return z, C_OVER_H0 * np.concatenate([[0.0], np.cumsum(0.5 * (e[1:] + e[:-1]) * 1e-3)])


def _directions(g, n, ra_deg, dec_deg):
    ra = _rand(g, n) * math.radians(ra_deg)
    s = _rand(g, n) * math.sin(math.radians(dec_deg))
    c = torch.sqrt(1.0 - s * s)
    return torch.stack([c * torch.cos(ra), c * torch.sin(ra), s], dim=1)


def _lightcone(g, n, ra_deg, dec_deg, z_mean=0.6, z_sd=0.15):
    """Points at comoving distances of a Gaussian n(z), observer at the origin."""
    z = (z_mean + z_sd * _normal(g, n)).clamp_(0.02, 2.9)
    zt, ct = _chi_table()
    ct = torch.from_numpy(ct).cuda()
    t = z / 1e-3
    k = t.long()
    chi = ct[k] + (ct[k + 1] - ct[k]) * (t - k)
    return _columns(g, _directions(g, n, ra_deg, dec_deg) * chi[:, None])


def _cap(g, n, half_deg, blobs):
    """Unit vectors in a cap around +x: uniform, or in blobs of 100 points of
    0.05 degrees."""
    m = n // 100 if blobs else n
    ct = 1.0 - _rand(g, m) * (1.0 - math.cos(math.radians(half_deg)))
    st, ph = torch.sqrt(1.0 - ct * ct), 2.0 * math.pi * _rand(g, m)
    v = torch.stack([ct, st * torch.cos(ph), st * torch.sin(ph)], dim=1)
    if blobs:
        v = v.repeat_interleave(100, dim=0) + math.radians(0.05) * _normal(g, m * 100, 3)
        if n > m * 100:
            v = torch.cat([v, v[: n - m * 100] + math.radians(0.05) * _normal(g, n - m * 100, 3)])
    return _columns(g, v / v.norm(dim=1, keepdim=True))


# ---------------------------------------------------------------------------
def _edges(c):
    if c.get("log"):
        return np.geomspace(c["r_max"] * 1e-2, c["r_max"], c["n1"] + 1)
    return np.linspace(0.0, c["r_max"], c["n1"] + 1)


def _rmu(c, los=cute.LOS_Z):
    return cute.Binning(cute.BIN_RMU, np.linspace(0.0, c["r_max"], c["n1"] + 1), np.linspace(0.0, 1.0, c["n2"] + 1), los=los)


def _theta_edges(c):
    t = np.deg2rad(c["theta_max"])
    if c.get("theta_min", 0.0) > 0.0:
        return np.geomspace(np.deg2rad(c["theta_min"]), t, c["n1"] + 1)
    return np.linspace(0.0, t, c["n1"] + 1)


def prepare(case, seed):
    c, p = case, case["path"]
    g, s = _gen(seed, 1), {"case": case}
    if p == "noalloc":
        s["bn"] = cute.Binning(cute.BIN_MONO, np.linspace(0.0, c["r_max"], c["n1"] + 1))
        s["grid"] = cute.build_grid(_box(g, c["n"], c["box"], 0.0, True), cute.GEOM_BOX_PERIODIC, box_size=c["box"],
                                    r_max=c["r_max"])
    elif p == "box":
        s["bn"] = cute.Binning(cute.BIN_MONO, _edges(c))
        s["d"] = _box(g, c["n"], c["box"], c["blob_frac"], True)
    elif p in ("rmu_dd", "rmu_xi"):
        s["bn"] = _rmu(c)
        s["d"] = _box(g, c["n"], c["box"], 1.0, False)
        if p == "rmu_xi":
            s["r"] = _box(_gen(seed, 2), c["n_rand"], c["box"], 0.0, False)
    elif p in ("sigmapi", "rmu_mid"):
        e = np.linspace(0.0, c["r_max"], c["n1"] + 1)
        s["bn"] = (cute.Binning(cute.BIN_SIGMAPI, e, np.linspace(0.0, c["r_max"], c["n2"] + 1), los=cute.LOS_MIDPOINT)
                   if p == "sigmapi" else _rmu(c, cute.LOS_MIDPOINT))
        sd = {"sigmapi": 0.15, "rmu_mid": 0.02}[p]
        s["d"] = _lightcone(g, c["n"], c["ra"], c["dec"], z_sd=sd)
        if c["n_rand"]:
            s["r"] = _lightcone(_gen(seed, 2), c["n_rand"], c["ra"], c["dec"], z_sd=sd)
    elif p == "theta":
        s["bn"] = cute.Binning(cute.BIN_THETA, _theta_edges(c))
        s["d"] = _cap(g, c["n"], c["half_angle"], True)
    elif p in ("wpix", "radial"):
        s["d"] = _columns(g, _directions(g, c["n"], 18.0, 18.0))
        s["zd"] = 0.5 + 0.1 * _rand(g, c["n"])
        if c["n_rand"]:
            g2 = _gen(seed, 2)
            s["r"] = _columns(g2, _directions(g2, c["n_rand"], 18.0, 18.0))
            s["zr"] = 0.5 + 0.1 * _rand(g2, c["n_rand"])
        s["bn"] = cute.Binning(cute.BIN_THETA, np.deg2rad(np.linspace(0.0, c.get("theta_max", 1.0), c["n1"] + 1)))
    elif p == "batch":
        k = np.arange(c["mocks"]) / max(1, c["mocks"] - 1)
        s["mocks"] = [_box(g, int(n), c["box"], 0.5, True)
                      for n in np.exp(np.log(c["n_lo"]) + k * np.log(c["n_hi"] / c["n_lo"]))]
        s["mono"] = cute.Binning(cute.BIN_MONO, np.linspace(0.0, 150.0, 31))
        s["bn"] = _rmu({"r_max": 200.0, "n1": 40, "n2": 50})
    else:
        s["bn"] = _rmu(c)
        s["d"] = _box(g, c["n"], c["box"], 0.5, True)
        m = c["side"]
        ix, iy = ((s["d"][k] * (m / c["box"])).long().clamp_(max=m - 1) for k in (0, 1))
        s["region"] = (iy * m + ix).to(torch.int32).contiguous()
    if "bn" in s:
        s["out"] = [torch.zeros(s["bn"].nbins, dtype=torch.int64, device="cuda") for _ in range(3)]
    return s


def run(state):
    s, c = state, state["case"]
    p, bn = c["path"], state.get("bn")
    if p == "noalloc":
        return cute.count_pairs_noalloc(s["grid"], None, bn, cute.PREC_FP32_EDGE, out=s["out"][0])
    if p == "box":
        g = cute.build_grid(s["d"], cute.GEOM_BOX_PERIODIC, box_size=c["box"], r_max=c["r_max"])
        dd = cute.count_pairs(g, None, bn, PREC[c["prec"]])
        g.close()
        return {"dd": dd, "xi": cute.xi_estimate(cute.EST_BOX, dd, None, None, c["n"], 0, bn, box_size=c["box"])}
    if p == "rmu_dd":
        g = cute.build_grid(s["d"], cute.GEOM_BOX_OPEN, r_max=c["r_max"])
        cute.count_pairs(g, None, bn, PREC[c["prec"]], out=s["out"][0])
        g.close()
        return s["out"][0]
    if p == "rmu_xi":
        gd = cute.build_grid(s["d"], cute.GEOM_BOX_OPEN, r_max=c["r_max"])
        gr = cute.build_grid(s["r"], cute.GEOM_BOX_OPEN, r_max=c["r_max"])
        dd = cute.count_pairs(gd, None, bn)
        dr = cute.count_pairs(gd, gr, bn)
        rr = cute.count_pairs(gr, None, bn)
        gd.close()
        gr.close()
        xi = cute.xi_estimate(cute.EST_LS, dd, dr, rr, c["n"], c["n_rand"], bn)
        return {"dd": dd, "dr": dr, "rr": rr, "xi": xi, "xi_l": cute.xi_multipoles(np.nan_to_num(xi), bn, (0, 2, 4))}
    if p in ("sigmapi", "rmu_mid"):
        reach = math.hypot(c["r_max"], c["r_max"]) if p == "sigmapi" else c["r_max"]
        gd = cute.build_grid(s["d"], cute.GEOM_BOX_OPEN, r_max=reach)
        gr = cute.build_grid(s["r"], cute.GEOM_BOX_OPEN, r_max=reach) if "r" in s else None
        cute.count_pairs(gd, gr, bn, out=s["out"][0])
        gd.close()
        if gr is not None:
            gr.close()
        return s["out"][0]
    if p == "theta":
        g = cute.build_grid(s["d"], cute.GEOM_SPHERE, r_max=float(bn.edges1[-1]))
        cute.count_pairs(g, None, bn, PREC[c["prec"]], out=s["out"][0])
        g.close()
        return s["out"][0]
    if p == "wpix":
        md = cute.build_pixel_map(s["d"], c["n_cth"], c["n_phi"], r_max=float(bn.edges1[-1]))
        mr = cute.build_pixel_map(s["r"], c["n_cth"], c["n_phi"], r_max=float(bn.edges1[-1]))
        dr = cute.count_pairs(md, mr, bn)
        md.close()
        mr.close()
        return dr
    if p == "radial":
        ap = math.radians(c["aperture"])
        gd = cute.build_grid(s["d"], cute.GEOM_SPHERE, r_max=ap)
        gr = cute.build_grid(s["r"], cute.GEOM_SPHERE, r_max=ap) if "r" in s else None
        n = cute.count_radial(gd, s["zd"], gr, s.get("zr"), ap, np.linspace(0.0, c["dz"], c["n1"] + 1))
        gd.close()
        if gr is not None:
            gr.close()
        return n
    if p == "batch":
        grids = [cute.build_grid(d, cute.GEOM_BOX_PERIODIC, box_size=c["box"], r_max=200.0) for d in s["mocks"]]
        items = [cute.BatchItem(g, None, b) for g in grids for b in (s["mono"], bn)]
        counts = cute.count_pairs_batched(items)
        for g in grids:
            g.close()
        return counts
    g = cute.build_grid(s["d"], cute.GEOM_BOX_PERIODIC, box_size=c["box"], r_max=c["r_max"])
    total, jack = cute.count_jackknife(g, s["region"], c["side"] ** 2, bn)
    g.close()
    return {"total": total, "jack": jack}


# ---------------------------------------------------------------------------
def _pairs(c):
    """Expected pairs in range (uniform catalogs plus the pairs inside blobs)."""
    p = c["path"]
    n, m = c.get("n", 0), c.get("n_rand", 0)
    if p in ("noalloc", "box", "rmu_dd", "rmu_xi", "jackknife"):
        v = 4.0 / 3.0 * math.pi * (c["r_max"] / c["box"]) ** 3
        blob = {"noalloc": 0.0, "box": c.get("blob_frac", 0.0), "jackknife": 0.5}.get(p, 1.0)
        dd = v * n * n / 2 + blob * n * 49.5
        return dd + (v * (n * m + m * m / 2) if p == "rmu_xi" else 0.0)
    if p == "batch":
        k = np.arange(c["mocks"]) / max(1, c["mocks"] - 1)
        ns = np.exp(np.log(c["n_lo"]) + k * np.log(c["n_hi"] / c["n_lo"]))
        return float(np.sum(ns * ns / 2) * 4.0 / 3.0 * math.pi * (0.15 ** 3 + 0.2 ** 3) + np.sum(ns) * 49.5)
    if p in ("sigmapi", "rmu_mid"):
        area = math.radians(c["ra"]) * math.sin(math.radians(c["dec"]))
        # 3-sigma depth of the n(z) at its mean distance (about 1580 Mpc/h, 2300 per unit z)
        vol = area * 1580.0 ** 2 * 2300.0 * (0.15 if p == "sigmapi" else 0.02) * math.sqrt(4 * math.pi)
        r = c["r_max"]
        v = (2 * math.pi * r ** 3 if p == "sigmapi" else 4.0 / 3.0 * math.pi * r ** 3) / vol
        return min(1.0, v) * (n * m if m else n * n / 2)
    if p == "theta":
        cap = 1.0 - math.cos(math.radians(c["half_angle"]))
        return min(1.0, (1.0 - math.cos(math.radians(c["theta_max"]))) / cap) * n * n / 2 + 49.5 * n
    area = math.radians(18.0) * math.sin(math.radians(18.0))
    t = math.radians(c.get("aperture", c.get("theta_max", 0.0)))
    share = min(1.0, 2 * math.pi * (1.0 - math.cos(t)) / area)
    if p == "wpix":
        px = area / (4 * math.pi) * c["n_cth"] * c["n_phi"]
        n, m = (px * (1.0 - math.exp(-k / px)) for k in (n, m))
    return share * (n * m if m else n * n / 2)


# operations of the formula for one pair in range: separation, bin, increment
OPS = {"noalloc": 14, "box": 14, "rmu_dd": 21, "rmu_xi": 21, "batch": 18, "jackknife": 42, "sigmapi": 40, "rmu_mid": 34,
       "theta": 16, "wpix": 16, "radial": 9}


def work(case):
    c, p = case, case["path"]
    if p == "batch":
        k = np.arange(c["mocks"]) / max(1, c["mocks"] - 1)
        pts = float(np.sum(np.exp(np.log(c["n_lo"]) + k * np.log(c["n_hi"] / c["n_lo"]))))
        bins = c["mocks"] * 2030
    else:
        pts = c["n"] + c.get("n_rand", 0)
        bins = c["n1"] * c.get("n2", 1) * (c["side"] ** 2 + 1 if p == "jackknife" else 3 if p == "rmu_xi" else 1)
    per_point = 32 if p == "radial" else 28 if p == "jackknife" else 24
    return {"bytes": per_point * pts + 8 * bins, "flops": OPS[p] * _pairs(c)}


# ---------------------------------------------------------------------------
def _count64(a, b, bn, box):
    """Brute-force counts of one catalog's pairs (b None) or of two catalogs,
    in float64, with torch."""
    auto = b is None
    q = a if auto else b
    e1 = torch.from_numpy(bn.edges1 ** 2).cuda()
    e2 = None if bn.edges2 is None else torch.from_numpy(bn.edges2 ** 2).cuda()
    n1, n2 = len(e1) - 1, 1 if e2 is None else len(e2) - 1
    tot = torch.zeros(n1 * n2, dtype=torch.int64, device="cuda")
    step = max(1, 40_000_000 // max(1, q.shape[0]))
    for i in range(0, a.shape[0], step):
        d = [(a[i:i + step, None, k] - q[None, :, k]) for k in range(3)]
        if box > 0:
            d = [torch.where(x > box / 2, x - box, torch.where(x < -box / 2, x + box, x)) for x in d]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        ok = (r2 >= e1[0]) & (r2 < e1[-1])
        if auto:
            j = torch.arange(q.shape[0], device="cuda")
            ok &= j[None, :] > torch.arange(i, min(i + step, a.shape[0]), device="cuda")[:, None]
        r2 = r2[ok]
        k = torch.bucketize(r2, e1, right=True) - 1
        if e2 is not None:
            m2 = torch.where(r2 > 0, d[2][ok] ** 2 / r2, torch.zeros_like(r2))
            k = k * n2 + (torch.bucketize(m2, e2, right=True) - 1).clamp_(0, n2 - 1)
        tot += torch.bincount(k, minlength=n1 * n2)
    return tot.cpu().numpy().astype(np.float64).reshape(bn.shape)


def exact(case, seed):
    """The correlation functions (the floating outputs) in 64 bits by brute
    force; the counts are whole numbers and have no rounding."""
    c, p = case, case["path"]
    if p not in ("box", "rmu_xi") or c["n"] * (c["n"] + c.get("n_rand", 0)) + c.get("n_rand", 0) ** 2 > 6e9:
        return None
    s = prepare(case, seed)
    bn = s["bn"]
    d = torch.stack(s["d"], dim=1)
    if p == "box":
        dd = _count64(d, None, bn, c["box"])
        e = bn.edges1
        shell = 4.0 / 3.0 * np.pi * (e[1:] ** 3 - e[:-1] ** 3) / c["box"] ** 3
        return {"dd": None, "xi": dd / (0.5 * c["n"] * (c["n"] - 1.0) * shell) - 1.0}
    r = torch.stack(s["r"], dim=1)
    dd, dr, rr = (_count64(x, y, bn, 0.0) for x, y in ((d, None), (d, r), (r, None)))
    nd, nr = float(c["n"]), float(c["n_rand"])
    with np.errstate(divide="ignore", invalid="ignore"):
        xi = (nr * (nr - 1) * dd - (nr - 1) * (nd - 1) * dr + nd * (nd - 1) * rr) / (nd * (nd - 1) * rr)
    xi[rr == 0] = np.nan
    m, w = bn.edges2, []
    for leg in ([1], [0, 0, 1], [0, 0, 0, 0, 1]):
        i = np.polynomial.legendre.legint(leg)
        w.append((2 * len(leg) - 1) * np.diff(np.polynomial.legendre.legval(m, i)))
    xi_l = np.stack([np.nan_to_num(xi) @ v for v in w])
    return {"dd": None, "dr": None, "rr": None, "xi": xi, "xi_l": xi_l}
