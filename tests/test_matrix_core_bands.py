"""CPU check of the rounding analysis behind the FP32_EDGE kernels whose
separations come from the matrix cores: |a|^2 + |b|^2 - 2 a.b with a and b the
points in the frame of the home tile, and the decisions made from it.

cute_fp32_count_constants (host only) reports what a count decides by. Here
the kernels' arithmetic is replayed exactly: every FP32 multiply, add and
subtract is an IEEE binary32 operation, every fused multiply-add (the matrix
instructions' steps among them) is rounded once from the exact rational value,
the squares and products formed in FP64 likewise, and the hardware 1/sqrt and
sqrt are replayed correctly rounded and perturbed by 2^-21 either way. The
pairs are adversarial: home points at the corners of their tile (the largest
|a|), separations within a few bands of the edges, coincident and nearly
coincident points, both far from the origin and in small length units. Checked:

* the error bound of the separations, with every term of it;
* every pair that FP32 certifies (in a bin, or out of range) agrees with the
  canonical FP64 classifier of the oracle and with the exact rational values;
* the positions in bin units and the predicates F of sigma and pi differ from
  the exact ones by less than what was removed from the bin;
* pairs far from every edge are decided in FP32.
"""
import math
from fractions import Fraction

import numpy as np
import pytest

import oracle
import paper_1210_1833_amd as cute
from test_midpoint_bands import F32, U32, U64, fma32, rsq32

B23 = F32(2.0 ** 23)
B231 = F32(2.0 ** 23 + 1.0)
BIG = 1e29


def fma64(a, b, c):
    return float(Fraction(float(a)) * Fraction(float(b)) + Fraction(float(c)))


def dot64(a, b):
    return fma64(a[2], b[2], fma64(a[1], b[1], float(a[0]) * float(b[0])))


def root32(x, pert):
    return F32(math.sqrt(float(x)) * (1.0 + pert)) if x >= 0 else F32(np.nan)


class Count:
    """The planned count of a grid and its tiles."""

    def __init__(self, case):
        self.case = case
        geom = getattr(cute, "GEOM_" + case.get("geom", "BOX_OPEN"))
        lo, hi = np.array(case["lo"], float), np.array(case["hi"], float)
        norm = case.get("norm", float(np.sqrt((np.maximum(abs(lo), abs(hi)) ** 2).sum())))
        self.k, self.b1, self.b2 = cute.fp32_count_constants(
            geom, case["n"], lo, hi, norm, case["bn"], box_size=case.get("L", 0.0), r_max=case["reach"],
            cell_size=case.get("cell", 0.0), radial=case.get("radial"))
        k = self.k
        self.lo, self.hi = lo, hi
        self.c = np.array([k["cx"], k["cy"], k["cz"]])
        self.cells = np.array([k["nx"], k["ny"], k["nz"]])
        self.o, self.a = np.array([k["ox"], k["oy"], k["oz"]]), np.array([k["ax"], k["ay"], k["az"]])

    def tile(self, rng):
        """A home tile: its box (lower and upper corner) and its origin's frame."""
        c0 = np.array([rng.integers(0, int(m)) for m in self.cells])
        w = min(int(self.k["max_w"]), int(self.cells[0] - c0[0]))
        c1 = int(c0[0]) + int(rng.integers(1, w + 1)) - 1
        lo = self.o + c0 * self.a
        hi = self.o + (np.array([c1, c0[1], c0[2]]) + 1) * self.a
        # the kernel's expressions, in its order
        mid = [self.k["ox"] + 0.5 * float(c0[0] + c1 + 1) * self.a[0] - self.c[0],
               self.k["oy"] + (float(c0[1]) + 0.5) * self.a[1] - self.c[1],
               self.k["oz"] + (float(c0[2]) + 0.5) * self.a[2] - self.c[2]]
        org = [F32(0.0) if self.cells[d] == 1 else F32(mid[d]) for d in range(3)]
        return np.maximum(lo, self.lo), np.minimum(hi, self.hi), org

    def frames(self, p, q, org, image):
        """a and b as the kernel forms them (image: periods between q and the
        neighbour in the home point's frame)."""
        Lf = F32(self.case.get("L", 0.0))
        hp = [F32(p[d] - self.c[d]) for d in range(3)]
        hq = [F32(q[d] - self.c[d]) for d in range(3)]
        a = [hp[d] - org[d] for d in range(3)]
        kx = [F32(0.0) - F32(image[d]) * Lf for d in range(3)]
        b = [(hq[d] - kx[d]) - org[d] for d in range(3)]
        return a, b


def separation(a, b):
    a2, b2 = dot64(a, a), dot64(b, b)
    m = [F32(-2.0) * x for x in a]
    v = fma32(m[0], b[0], F32(b2))
    v = fma32(m[1], b[1], v)
    v = fma32(m[2], b[2], v)
    return fma32(F32(a2), F32(1.0), v), a2, b2


def clamped(ts, e1a, top):
    e = fma32(ts, e1a, B23)
    return int(top) if not e >= 0 else int(min(max(float(e) - 2.0 ** 23, 0.0), top))


def in_band(v, b):
    return bool(b[0] <= v <= b[1])


def midpoint_tile(cn, org):
    """L0 and the tile's own constants (FP32, in the kernel's order)."""
    k, u = cn.k, F32(2.0 ** -24)
    L = [F32(2.0 * (cn.c[d] + float(org[d]))) for d in range(3)]
    l0 = F32(math.sqrt(float(F32(dot64(L, L)))))
    M = F32(k["M"])
    Lx = fma32(l0, F32(1.00001), M)
    esl = F32(1.001) * u * (Lx * M + M * M)
    ell = F32(1.011) * u * (F32(3.0) * Lx * Lx + F32(2.0) * Lx * M + F32(9.1) * M * M)
    if cn.case["kind"] == "sp":
        t = F32(k["K1"]) * Lx + F32(k["K0"]) + F32(k["TR"]) * ell + F32(k["2R"]) * Lx * esl + esl * esl
        return L, max(F32(1.1) * t, F32(k["Tmin"])), None, None
    lmin = l0 * F32(0.99999) - M
    i = F32(1.0) / lmin
    fe, N = F32(k["fe"]), F32(k["N"])
    d0 = N * (F32(2.0) * fe * i + F32(0.5) * ell * i * i)
    d1 = N * esl * i
    ok = lmin > F32(0.05) * M and lmin > F32(16.0) * fe and d0 < F32(0.2)
    return L, F32(1.0 if ok else -1.0), F32(k["muB0"]) - F32(1.001) * d0, F32(k["muB1"]) - F32(1.001) * d1


def decide(cn, v, a, b, a2, b2, org, pert, zz):
    """(certified bin or None, certainly out, values) of the kernel."""
    k, kind = cn.k, cn.case["kind"]
    e1a, s1, e2a, s2 = (F32(k[n]) for n in ("e1a", "s1", "e2a", "s2"))
    n2 = cn.b2.shape[0] - 1
    lt = bool(v < F32(k["skip32"]))
    low = bool(v < F32(k["out_lo"])) if kind != "sp" else False
    if kind in ("mono", "theta"):
        if kind == "theta":
            ch = root32(v, pert)
            th = fma32(ch * v, F32(1.0 / 24.0), ch) if v >= 0 else F32(np.nan)
            ts = th + s1
            if int(k["est"]) & 1:
                ts = F32(np.nan) if not v > 0 else F32(math.log2(float(th))) + s1
        elif int(k["est"]) & 1:
            ts = F32(np.nan) if not v > 0 else F32(math.log2(float(v))) + s1
        else:
            ts = fma32(v, rsq32(v, pert), s1) if v > 0 else F32(np.nan)
        kb = clamped(ts, e1a, k["top1"]) if np.isfinite(ts) else int(k["top1"])
        # (any estimate may be taken: the band alone certifies)
        hits = [j for j in range(len(cn.b1) - 1) if in_band(v, cn.b1[j])]
        assert len(hits) <= 1
        return (kb if in_band(v, cn.b1[kb]) else None), not lt or low, {}
    if kind == "radial":
        A = k["rdA"]
        al, w = F32(zz[0] * A), F32(zz[1] * A)
        half = fma32(F32(-3.5 * 2.0 ** -24), abs(al) + abs(w), F32(k["rB0"]))
        d = fma32(al, F32(1.0), -w)
        ts = abs(d) + s1
        e = ts + B231
        sure = abs(ts + (B231 - e)) <= half and lt
        j = int(float(e) - float(B231))
        inside = j < len(cn.b1) - 1 and (not k["rdLow"] or j >= 0)
        cert = j if sure and inside and v <= F32(k["rdIn"]) else None
        return cert, not lt or (sure and not inside), dict(ts=ts, half=half)
    if not v > 0:
        return None, not lt or low, {}
    rinv = rsq32(v, pert)
    if kind == "rmu":
        dz = fma32(F32(-2.0) * a[2], F32(-0.5), -b[2])
        d0, d1, mt = F32(k["muB0"]), F32(k["muB1"]), None
    else:
        L, mt, d0, d1 = midpoint_tile(cn, org)
        al = F32(dot64(L, a) + a2)
        beta = dot64(L, b) + b2
        sl = fma32(al, F32(1.0), F32(-beta))
        ss = fma32(al, F32(2.0), F32(fma64(2.0, beta, dot64(L, L))))
        ll = ss - v
        if kind == "sp":
            sl2 = sl * sl
            c2 = fma32(v, ll, -sl2)
            nt = -mt
            ins = [abs(fma32(x[0], ll, c2)) <= fma32(x[1], ll, nt) for x in cn.b1]
            inp = [abs(fma32(x[0], ll, sl2)) <= fma32(x[1], ll, nt) for x in cn.b2]
            hit = [(i, j) for i in range(len(ins)) for j in range(len(inp)) if lt and ins[i] and inp[j]]
            assert len(hit) <= 1
            past = [h for h in hit if h[0] == len(ins) - 1 or h[1] == len(inp) - 1]
            out = not lt or bool(past)
            if k["low"]:
                out = out or fma32(F32(k["wsbot"]), ll, c2) <= nt or fma32(F32(k["wpbot"]), ll, sl2) <= nt
            cert = hit[0][0] * n2 + hit[0][1] if hit and not past else None
            return cert, out, dict(ll=ll, c2=c2, sl2=sl2, t=mt)
        if mt < 0:
            return None, not lt, {}
        dz = sl * rsq32(ll, pert)
    ts = fma32(v, rinv, s1) if not int(k["est"]) & 1 else F32(math.log2(float(v))) + s1
    ts2 = fma32(abs(dz), rinv, s2)
    if int(k["est"]) & 2:
        em = fma32(ts2, e2a, B231)
        half = fma32(fma32(F32(k["muB2"]), rinv, d1), rinv, d0)
        inm = abs(fma32(ts2, e2a, B231 - em)) <= half
        km = int(float(em) - float(B231))
        if int(k["est"]) & 1:
            kr = clamped(ts, e1a, k["top1"])
            inr = in_band(v, cn.b1[kr])
        else:
            er = fma32(ts, e1a, B231)
            inr = abs(fma32(ts, e1a, B231 - er)) <= F32(k["rB0"])
            kr = int(float(er) - float(B231))
        cert = kr * n2 + km if inr and inm and lt else None
        return cert, not lt or low, dict(ts=ts, ts2=ts2, half=half)
    raise AssertionError("r-mu with band tables has no matrix-core kernel")


LIN, MU = np.linspace(0.0, 200.0, 41), np.arange(51) / 50.0
RMU, MONO, SP, THETA = cute.BIN_RMU, cute.BIN_MONO, cute.BIN_SIGMAPI, cute.BIN_THETA
MID = cute.LOS_MIDPOINT
SURVEY = dict(lo=[700.0, -400.0, 0.0], hi=[2100.0, 900.0, 1000.0])


def case(kind, e1, e2=None, mid=False, radial=None, **more):
    name = {"mono": "MONO", "rmu": "RMU", "mid": "RMU", "sp": "SIGMAPI", "theta": "THETA", "radial": "THETA"}[kind]
    e1 = np.asarray(e1, float)
    bn = cute.Binning(getattr(cute, "BIN_" + name), e1, e2, los=MID if mid else cute.LOS_Z)
    ob = oracle.Binning(getattr(oracle, name), e1, e2, los=oracle.LOS_MID if mid else oracle.LOS_Z)
    r = float(np.hypot(e1[-1], e2[-1]) * (1 + 1e-12)) if name == "SIGMAPI" else float(e1[-1])
    return dict(kind=kind, bn=bn, ob=ob, e1=e1, e2=e2, reach=r, mid=mid, radial=radial, **more)


BOX = dict(lo=[0.0] * 3, hi=[2000.0] * 3)
CASES = {
    "rmu_bench": case("rmu", LIN, MU, n=1000000, **BOX),
    "rmu_far": case("rmu", LIN[:31], MU[::2], n=100000, lo=[2e4, -3e4, 1e4], hi=[2.3e4, -2.7e4, 1.3e4]),
    "rmu_coarse": case("rmu", LIN[:13], MU[::5], n=300000, cell=180.0, **BOX),
    "rmu_log": case("rmu", np.geomspace(0.1, 150.0, 25), MU, n=500000, **BOX),
    "rmu_kpc": case("rmu", LIN * 1e3, MU, n=1000000, lo=[0.0] * 3, hi=[2e6] * 3),
    "mono": case("mono", LIN, n=1000000, **BOX),
    "mono_up_coarse": case("mono", LIN[3:20], n=300000, cell=150.0, **BOX),
    "mono_log_kpc": case("mono", np.geomspace(1e-2, 1.5e5, 30), n=200000, lo=[0.0] * 3, hi=[2e6] * 3),
    "mono_periodic": case("mono", LIN[:31], n=100000, geom="BOX_PERIODIC", L=1000.0, lo=[0.0] * 3, hi=[999.99] * 3),
    # a thin slab: one cell along z, whose points span far less than the others
    "mono_slab": case("mono", LIN[:13], n=100000, lo=[0.0] * 3, hi=[2000.0, 2000.0, 20.0]),
    "rmu_slab": case("rmu", LIN[:13], MU[::5], n=100000, lo=[0.0] * 3, hi=[2000.0, 2000.0, 20.0]),
    "sp": case("sp", np.linspace(0.0, 150.0, 31), np.linspace(0.0, 150.0, 31), mid=True, n=3000000, **SURVEY),
    "sp_up": case("sp", np.linspace(3.0, 80.0, 21), np.linspace(3.0, 60.0, 21), mid=True, n=300000, **SURVEY),
    "mid": case("mid", LIN, MU, mid=True, n=1000000, **SURVEY),
    "mid_log": case("mid", np.geomspace(0.5, 120.0, 21), MU[::2], mid=True, n=300000, **SURVEY),
    "mid_near": case("mid", np.linspace(0.0, 40.0, 11), MU[::5], mid=True, n=300000, lo=[-300.0] * 3, hi=[300.0] * 3),
    "theta": case("theta", np.deg2rad(np.linspace(0.0, 5.0, 21)), n=500000, geom="SPHERE", lo=[0.2, -0.5, -0.4],
                  hi=[1.0, 0.5, 0.6], norm=1.0),
    "theta_log": case("theta", np.deg2rad(np.geomspace(1e-3, 10.0, 31)), n=2000000, geom="SPHERE",
                      lo=[0.2, -0.5, 0.3], hi=[0.9, 0.5, 0.98], norm=1.0),
    "radial": case("radial", [0.0, math.radians(1.0)], n=300000, geom="SPHERE", lo=[0.2, -0.5, -0.4],
                   hi=[1.0, 0.5, 0.6], norm=1.0, radial=np.linspace(0.0, 0.1, 101)),
    "radial_chi": case("radial", [0.0, math.radians(0.5)], n=300000, geom="SPHERE", lo=[0.2, -0.5, -0.4],
                       hi=[1.0, 0.5, 0.6], norm=1.0, radial=np.linspace(5.0, 150.0, 59)),
}


def separation_size(rng, c, edges):
    """Near an edge (from some bands to far inside one), tiny, zero, or anywhere."""
    e = edges[rng.integers(0, len(edges))]
    pick = rng.integers(8)
    if pick < 4:
        return e * (1.0 + rng.choice([-1.0, 1.0]) * 10.0 ** rng.uniform(-8.0, -3.0))
    if pick == 4:
        return c["reach"] * 10.0 ** rng.uniform(-7.0, -3.0)
    if pick == 5:
        return 0.0 if rng.integers(2) else e
    return rng.uniform(0.0, c["reach"] * 1.05)


def draw_pair(rng, cn):
    """(p, q, origin of the tile's frame, images)."""
    c = cn.case
    for _ in range(200):
        if c.get("geom") == "SPHERE":
            k = cn.k
            iz, ip = int(rng.integers(0, int(k["ny"]))), int(rng.integers(0, int(k["nx"])))
            w = int(rng.integers(1, int(min(k["max_w"], k["nx"])) + 1))

            def point():
                z = k["oy"] + (iz + rng.choice([1e-9, rng.uniform(), 1 - 1e-9])) * k["ay"]
                f = (ip + rng.choice([1e-9, rng.uniform(), 1 - 1e-9]) * w) * k["ax"]
                s = math.sqrt(max(0.0, 1.0 - z * z))
                return np.array([s * math.cos(f), s * math.sin(f), z])
            p, o = point(), point()
            org = [F32(x) for x in o]
            t = separation_size(rng, c, c["e1"])
            e = np.cross(p, rng.normal(size=3))
            e /= np.linalg.norm(e)
            q = p * math.cos(t) + e * math.sin(t)
            q = q / np.linalg.norm(q) if t else p.copy()
            return p, q, org, (0, 0, 0)
        lo, hi, org = cn.tile(rng)
        f = rng.uniform(size=3)
        f[rng.uniform(size=3) < 0.5] = rng.choice([0.0, 1.0])
        p = np.clip(lo + f * (hi - lo), cn.lo, cn.hi)
        e = rng.normal(size=3)
        if c["kind"] in ("mono",):
            e *= separation_size(rng, c, c["e1"]) / np.linalg.norm(e)
        else:
            n = np.array([0.0, 0.0, 1.0]) if not c["mid"] else p / max(np.linalg.norm(p), 1e-300)
            e -= n * (e @ n)
            e /= np.linalg.norm(e)
            if c["kind"] == "sp":
                e = e * separation_size(rng, c, c["e1"]) + n * rng.choice([-1, 1]) * separation_size(rng, c, c["e2"])
            else:
                mu = c["e2"][rng.integers(0, len(c["e2"]))] * (1 + rng.choice([-1, 1]) * 10.0 ** rng.uniform(-8, -3))
                mu = min(max(mu if rng.integers(2) else rng.uniform(), 0.0), 1.0)
                r = separation_size(rng, c, c["e1"])
                e = r * (math.sqrt(1 - mu * mu) * e + mu * rng.choice([-1, 1]) * n)
        q, image = p + e, (0, 0, 0)
        if c.get("geom") == "BOX_PERIODIC":
            L = c["L"]
            image = tuple(int(math.floor(x / L)) for x in q)
            q = np.array([x - i * L for x, i in zip(q, image)])
        if np.all(q >= cn.lo) and np.all(q <= cn.hi):
            return p, q, org, image
    raise AssertionError("no pair found inside the box")


@pytest.mark.parametrize("name", sorted(CASES))
def test_decisions_on_adversarial_pairs(name):
    c = CASES[name]
    rng = np.random.default_rng(sorted(CASES).index(name) + 900)
    cn = Count(c)
    k = cn.k
    assert k["path"] == 2.0, k
    assert k["out_lo"] == -math.inf or k["out_lo"] > 0.0 or c["kind"] == "sp"
    ec, ec64, ta, s3 = k["ec"], k["ec64"], k["ta"], math.sqrt(3.0)
    n2 = cn.b2.shape[0] - 1
    E1 = [Fraction(float(x)) for x in c["e1"]]
    M2 = [Fraction(float(x * x)) for x in c["e2"]] if c["e2"] is not None else None
    S2 = [x * x for x in E1]
    zmax = 0.6 if c["radial"] is not None and c["radial"][-1] < 1.0 else 2300.0
    decided = far = far_decided = 0
    worst = {"v": 0.0, "a": 0.0, "1": 0.0, "2": 0.0}
    for i in range(900):
        p, q, org, image = draw_pair(rng, cn)
        zz = None
        L = Fraction(c.get("L", 0.0))
        s_ex = [Fraction(float(x)) - Fraction(float(y)) - m * L for x, y, m in zip(p, q, image)]
        l_ex = [Fraction(float(x)) + Fraction(float(y)) for x, y in zip(p, q)]
        r2 = sum(x * x for x in s_ex)
        r = math.sqrt(float(r2))
        if c["kind"] == "radial":
            z0 = rng.uniform(0.3, 1.0) * zmax
            d = separation_size(rng, dict(reach=c["radial"][-1]), c["radial"])
            zz = (z0, z0 + d if rng.integers(2) else max(z0 - d, 0.0))
            dz = abs(zz[0] - zz[1])
            ap2 = (2.0 * math.sin(0.5 * c["e1"][-1])) ** 2
            dd = [x - y for x, y in zip(p, q)]
            inside = fma64(dd[2], dd[2], fma64(dd[1], dd[1], dd[0] * dd[0])) < ap2
            j = int(np.searchsorted(c["radial"], dz, side="right")) - 1
            canon = j if inside and 0 <= j < len(c["radial"]) - 1 else -1
        elif image != (0, 0, 0) or c.get("geom") == "BOX_PERIODIC":
            canon = -1 if r2 >= S2[-1] else max(j for j in range(len(S2) - 1) if S2[j] <= r2)
            if min(abs(r2 - x) for x in S2) < Fraction(1, 10 ** 11) * S2[-1]:
                canon = None   # (the FP64 minimum image may round to either side)
        else:
            canon = oracle.classify(p, q, c["ob"])
        for pert in (-2.0 ** -21, 0.0, 2.0 ** -21):
            a, b = cn.frames(p, q, org, image)
            v, a2, b2 = separation(a, b)
            cert, out, w = decide(cn, v, a, b, a2, b2, org, pert, zz)
            if cert is not None and canon is not None:
                assert canon == cert, (i, canon, cert, float(r2))
                assert not out
            if out and canon is not None:
                assert canon == -1, (i, canon, float(r2), float(v))
            if pert != 0.0:
                continue
            # the reach of a tile, and the bound of the separation
            na = math.sqrt(a2)
            worst["a"] = max(worst["a"], na / ta)
            es = max(abs(Fraction(float(x)) - Fraction(float(y)) - z) for x, y, z in zip(a, b, s_ex))
            assert es <= Fraction(ec), (i, float(es), ec)
            if r <= 1.02 * c["reach"]:
                m = 2 * ta + r + 2 * s3 * ec
                bound = 2 * s3 * r * ec + 3 * ec * ec + 3.01 * U32 * (r + s3 * ec) ** 2 + 5.1 * U32 * m * m
                worst["v"] = max(worst["v"], abs(float(Fraction(float(v)) - r2)) / bound)
            done = cert is not None or out
            decided += done
            # how far the values are from the exact ones, against what the
            # bands allow, and whether pairs far from every edge are decided
            if c["kind"] in ("rmu", "mid") and int(k["est"]) & 2 and w and r2 > 0 and r2 < S2[-1]:
                if c["kind"] == "rmu":
                    mu = abs(float(s_ex[2])) / r
                else:
                    ll = sum(x * x for x in l_ex)
                    mu = abs(float(sum(x * y for x, y in zip(s_ex, l_ex)))) / (r * math.sqrt(float(ll)))
                x2, x2e = float(w["ts2"]) * k["e2a"], (mu + k["s2"]) * k["e2a"]
                room = 0.5 - float(w["half"])
                if room < 0.5:
                    worst["2"] = max(worst["2"], abs(x2 - x2e) / room)
                off = 0.5 - abs(x2e - round(x2e))
                if int(k["est"]) & 1:
                    continue
                x1, x1e = float(w["ts"]) * k["e1a"], (r + k["s1"]) * k["e1a"]
                if r > 0.5 * c["e1"][1]:
                    worst["1"] = max(worst["1"], abs(x1 - x1e) / (0.5 - k["rB0"]))
                if min(off / room, (0.5 - abs(x1e - round(x1e))) / (0.5 - k["rB0"])) > 4 and mu < 1 - 1e-6:
                    far += 1
                    far_decided += done
            elif c["kind"] == "sp" and w and r < c["reach"]:
                ll = float(sum(x * x for x in l_ex))
                sl = sum(x * y for x, y in zip(s_ex, l_ex))
                pi2 = float(sl * sl / sum(x * x for x in l_ex))
                sig2 = float(r2) - pi2
                t = float(w["t"]) / float(w["ll"])
                margin = []
                for val, got, edges, bt, key in ((sig2, w["c2"], c["e1"], cn.b1, "1"), (pi2, w["sl2"], c["e2"], cn.b2, "2")):
                    j = int(np.argmin(np.abs(edges ** 2 - val)))
                    if j == 0:
                        room = -float(bt[0][0]) - float(bt[0][1]) - edges[0] ** 2 if edges[0] > 0 else np.inf
                    else:
                        room = edges[j] ** 2 - (-float(bt[j - 1][0]) + float(bt[j - 1][1]))
                    if np.isfinite(room):
                        worst[key] = max(worst[key], abs(float(got) / float(w["ll"]) - val) / (room + t))
                        margin.append(abs(val - edges[j] ** 2) / (room + t))
                if margin and min(margin) > 4:
                    far += 1
                    far_decided += done
            elif c["kind"] == "radial" and w and r2 < Fraction(float(k["rdIn"])) * Fraction(99, 100):
                x, xe = float(w["ts"]), dz * k["rdA"] + k["s1"]
                room = 0.5 - float(w["half"])
                worst["1"] = max(worst["1"], abs(x - xe) / room)
                if 0.5 - abs(xe - round(xe)) > 4 * room:
                    far += 1
                    far_decided += done
            elif c["kind"] in ("mono", "theta"):
                T = [float(x) ** 2 for x in c["e1"]] if c["kind"] == "mono" else [
                    (2.0 * math.sin(0.5 * float(x))) ** 2 for x in c["e1"]]
                if r2 > 0 and r <= c["reach"]:
                    m = 2 * ta + r
                    # (a separation inside its own error may come out negative)
                    gap = min(abs(float(r2) - x) for x in T + [0.0]) / (1.5 * (2 * s3 * r * ec + 5.1 * U32 * m * m))
                    if gap > 4:
                        far += 1
                        far_decided += done
    print(name, "decided", decided, "far", far, {x: round(y, 3) for x, y in worst.items()})
    assert worst["v"] <= 1.0 and worst["1"] <= 1.0 and worst["2"] <= 1.0 and worst["a"] <= 1.0, worst
    assert far_decided == far, (far, far_decided)
    # (most pairs lie within a few bands of an edge by construction)
    assert decided > 100


@pytest.mark.parametrize("lo,hi", [([1600.0] * 3, [2600.0] * 3), ([3000.0, -200.0, 2500.0], [4000.0, 800.0, 3500.0])])
def test_midpoint_line_of_sight_of_the_component_form(lo, hi):
    # r bins so fine in a tile so large that r-mu is counted with component-wise
    # separations: its line of sight l = h + ((q - c) + 2 c) has roundings of
    # its own, which the planned bound of l covers
    c = case("mid", np.linspace(0.0, 120.0, 1001), np.linspace(0.0, 1.0, 5), mid=True, n=200000, cell=60.0, lo=lo, hi=hi)
    cn = Count(c)
    assert cn.k["path"] == 1.0, cn.k
    rng = np.random.default_rng(5)
    pts = rng.uniform(lo, hi, (200000, 3))
    q = pts + rng.uniform(-60.0, 60.0, pts.shape)
    hp, hq = (pts - cn.c).astype(np.float32), (q - cn.c).astype(np.float32)
    l32 = hp + (hq + (2.0 * cn.c).astype(np.float32))
    # (the exact sum of two doubles: l32 - p is exact to far below the bound)
    err = np.abs((l32.astype(np.float64) - pts) - q).max()
    print("worst |l32 - l|", err, "bound", cn.k["el"])
    assert err <= cn.k["el"]


@pytest.mark.parametrize("path,c", [
    # a tile's frame as large as the separations, and bins as fine as its error
    (1, case("theta", np.deg2rad(np.linspace(0.0, 30.0, 257)), n=300000, geom="SPHERE", lo=[0.9, 0.0, 0.0],
             hi=[1.0, 0.31, 0.31], norm=1.0, cell=6.0)),
    (2, case("theta", np.deg2rad(np.linspace(0.0, 30.0, 257)), n=300000, geom="SPHERE", lo=[0.9, 0.0, 0.0],
             hi=[1.0, 0.31, 0.31], norm=1.0)),
    (1, case("rmu", np.linspace(0.0, 60.0, 101), MU[::5], n=100000, cell=300.0, lo=[0.0] * 3, hi=[500.0] * 3)),
    (2, case("rmu", np.linspace(0.0, 60.0, 101), MU[::5], n=100000, lo=[0.0] * 3, hi=[500.0] * 3)),
    # general r or mu edges
    (1, case("rmu", LIN[4:], MU, n=500000, **BOX)),
    (1, case("rmu", LIN, MU ** 2, n=500000, **BOX)),
    # lengths past the range of the matrix cores, and of FP32 squares
    (2, case("mid", LIN, MU, mid=True, n=1000000, **SURVEY)),
    (1, case("mid", LIN * 2e4, MU, mid=True, n=1000000, lo=[x * 2e4 for x in SURVEY["lo"]],
             hi=[x * 2e4 for x in SURVEY["hi"]])),
    (1, case("mid", LIN * 1e6, MU, mid=True, n=1000000, lo=[x * 1e6 for x in SURVEY["lo"]],
             hi=[x * 1e6 for x in SURVEY["hi"]])),
    (0, case("mid", LIN * 1e9, MU, mid=True, n=1000000, lo=[x * 1e9 for x in SURVEY["lo"]],
             hi=[x * 1e9 for x in SURVEY["hi"]])),
    (1, case("mono", LIN * 1e12, n=1000000, lo=[0.0] * 3, hi=[2e15] * 3)),
    (0, case("mono", LIN * 1e15, n=1000000, lo=[0.0] * 3, hi=[2e18] * 3)),
    # radial counts: the matrix cores unless most pairs in the aperture are near it
    (2, case("radial", [0.0, math.radians(1.0)], n=100000, geom="SPHERE", lo=[0.9, 0.0, 0.0], hi=[1.0, 0.31, 0.31],
             norm=1.0, radial=np.linspace(0.0, 0.1, 101), cell=6.0)),
    (0, case("radial", [0.0, math.radians(0.5)], n=100000, geom="SPHERE", lo=[0.999, 0.0, 0.0], hi=[1.0, 0.0175, 0.0175],
             norm=1.0, radial=np.linspace(0.0, 0.1, 101), cell=6.0)),
])
def test_form_of_the_separations(path, c):
    assert Count(c).k["path"] == path


def test_reach_of_a_slabs_tiles():
    # the reach is that of the tile's own box: with the largest half extent in
    # place of the slab's, 1000 here, r-mu counts lost the matrix cores
    for name in ("mono_slab", "rmu_slab"):
        k = Count(CASES[name]).k
        assert k["nz"] == 1.0 and k["path"] == 2.0
        assert k["ta"] <= 0.51 * math.sqrt((k["max_w"] * k["ax"]) ** 2 + k["ay"] ** 2 + k["az"] ** 2)


@pytest.mark.parametrize("cell", [0.0, 300.0])
def test_largest_separation_of_a_decided_sigma_pi_pair(cell):
    # a pair is decided when v < skip32, and v may be below |s|^2 by its error
    c = case("sp", np.linspace(0.0, 20.0, 5), np.linspace(0.0, 20.0, 5), mid=True, n=300000, cell=cell, **SURVEY)
    k = Count(c).k
    assert k["path"] == 2.0
    R = 0.5 * k["2R"]
    err = 5.1 * U32 * (2 * k["ta"] + R) ** 2 + 2 * math.sqrt(3.0) * R * k["ec"]
    assert R * R >= k["skip32"] + err
