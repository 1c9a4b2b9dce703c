"""The work that users of the library have it do, as timed cases.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` makes what a caller holds before the call (Year Event Table, loaded
portfolio, or the host description of one), ``run`` is one pass through the
public entry points, ``work`` what that pass cannot do without, and ``exact``
its results in 64 bits by plain torch.

Kinds of case (``"kind"``):

* ``run``: one ``Ara.run`` of a loaded portfolio over a resident YET, with or
  without secondary uncertainty, with or without the occurrence view.
* ``batch``: one ``Ara.run_batch`` of several loaded portfolios.
* ``price``: what a request for a new portfolio costs: ``load_portfolio``,
  ``run`` over a part of the YET, ``free_portfolio``.
* ``metrics``: PML / TVaR and the exceedance curve of a Year Loss Table.

Row laws (``"law"``), all with lognormal means:

* ``single``: sigma_I = mean / 2, exposure = 4 mean (every row one Beta shape);
* ``mix``: sigma_I = sigma_C = mean / 4, the two-normal mix;
* ``varied``: sigma_I = mean U(0.15, 0.9), exposure = mean U(1.5, 10), every
  row its own shape, as in loss tables taken from catastrophe models;
* ``capped``: ``single`` with 30 % of the rows at sigma_I = 3 mean, above the
  largest standard deviation a Beta can have.
"""
from __future__ import annotations

import math
from dataclasses import dataclass
from typing import List

import numpy as np
import torch

INF = float("inf")
LIMITS = {"elt_r": 1e6, "elt_l": 5e7, "occ_r": 1e7, "occ_l": 2e8, "agg_r": 5e7, "agg_l": 1e9}
RETURN_PERIODS = (2.0, 5.0, 10.0, 25.0, 50.0, 100.0, 250.0, 500.0, 1000.0)


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _run(name, **kw):
    c = {"name": name, "kind": "run", "su": True, "law": "single", "trials": 1000, "lam": 1000.0,
         "catalogue": 100_000, "layers": 1, "elts": 16, "rows": 20_000, "scale": 1.0,
         "fit": False, "terms": "fixed", "sum_mode": "kahan32", "ylt": "f32", "view": False,
         "keying": 0}
    c.update(kw)
    return c


def listed():
    return [
        # the benchmark's analysis: a layer of 16 tables over a million simulated years
        _run("su_full", trials=1_000_000),
        # an interactive what-if: a small book over ten thousand years
        _run("su_small", trials=10_000, lam=100.0, catalogue=10_000, elts=3, rows=2_000, scale=0.1),
        # correlated and independent uncertainty together, as the method states it
        _run("su_mix", trials=40_003, law="mix"),
        # every row with its own shape, as vendors deliver loss tables
        _run("su_varied", trials=20_011, law="varied"),
        # tables with some rows of implausibly large uncertainty
        _run("su_capped", trials=20_011, law="capped"),
        # where each occurrence's loss goes: the per-occurrence report of a quarter million years
        _run("su_view", trials=250_000, view=True),
        # mean losses only, over the whole YET: the quick look before the full analysis
        _run("pu_full", su=False, trials=1_000_000),
        # mean losses over a fine catalogue whose tables exceed the on-chip memory
        _run("pu_catalogue", su=False, trials=300_007, catalogue=1_000_000),
        # a programme of eight layers, FP64 sums and FP64 Year Loss Tables
        _run("pu_layers", su=False, trials=100_003, layers=8, elts=18, terms="random",
             sum_mode="f64", ylt="f64"),
        # a night's batch of treaties, each of several layers, over a part of the YET
        {"name": "batch", "kind": "batch", "su": True, "law": "single", "trials": 25_000,
         "lam": 1000.0, "catalogue": 100_000, "portfolios": 4, "layers": 5, "elts": 16,
         "rows": 12_000, "scale": 1.0, "sum_mode": "kahan32", "ylt": "f32", "keying": 0},
        # one pricing request of the serving workload: a new portfolio, a part of the YET
        {"name": "price", "kind": "price", "su": True, "law": "single", "trials": 50_021,
         "lam": 1000.0, "catalogue": 100_000, "layers": 4, "elts": 16, "rows": 12_000,
         "scale": 1.0, "terms": "random", "sum_mode": "kahan32", "ylt": "f32", "keying": 0},
        # the risk report from a Year Loss Table: nine return periods and the whole curve
        {"name": "metrics", "kind": "metrics", "trials": 1_000_000, "ylt": "f32", "periods": 9},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  Each kind keeps the ranges of its listed cases: trials,
    occurrences, catalogue, tables and rows spread over their logarithm."""
    pick = rng.choice(["su", "su", "mix", "varied", "capped", "view", "pu", "pu", "layers",
                       "batch", "price", "metrics"])
    lam = float(_log_int(rng, 60, 1200))
    cat = rng.choice([10_000, 30_011, 100_000, 250_007])
    elts = rng.randint(2, 24)
    rows = min(cat // 3, _log_int(rng, 1_000, 30_000))
    scale = 0.1 if lam < 300 else 1.0
    common = {"lam": lam, "catalogue": cat, "elts": elts, "rows": rows, "scale": scale,
              "fit": True}
    if pick == "metrics":
        return {"kind": "metrics", "trials": _log_int(rng, 5_000, 1_000_000),
                "ylt": rng.choice(["f32", "f64"]), "periods": rng.randint(1, 9)}
    if pick == "batch":
        return {"kind": "batch", "su": rng.random() < 0.7, "law": "single",
                "trials": _log_int(rng, 2_000, 25_000), "portfolios": rng.randint(2, 5),
                "layers": rng.randint(1, 4), "sum_mode": "kahan32", "ylt": "f32",
                "keying": rng.choice([0, 1]), **dict(common, elts=rng.randint(2, 16))}
    if pick == "price":
        return {"kind": "price", "su": rng.random() < 0.7,
                "law": rng.choice(["single", "varied"]), "trials": _log_int(rng, 2_000, 20_000),
                "layers": rng.randint(1, 5), "terms": "random", "sum_mode": "kahan32",
                "ylt": "f32", "keying": 0, **dict(common, elts=rng.randint(2, 16))}
    c = _run("", **common)
    del c["name"]
    if pick in ("su", "pu"):
        c.update(su=pick == "su", trials=_log_int(rng, 1_000, 500_000),
                 sum_mode=rng.choice(["kahan32", "kahan32", "naive32", "f64"]),
                 catalogue=rng.choice([cat, cat, 1_000_000]), keying=rng.choice([0, 0, 1]))
    elif pick == "mix":
        c.update(law="mix", trials=_log_int(rng, 1_000, 40_000), keying=rng.choice([0, 1]))
    elif pick in ("varied", "capped"):
        c.update(law=pick, trials=_log_int(rng, 1_000, 20_000))
    elif pick == "view":
        c.update(su=rng.random() < 0.5, view=True, trials=_log_int(rng, 1_000, 250_000),
                 layers=rng.randint(1, 2))
    else:
        c.update(su=False, layers=rng.randint(2, 8), terms="random",
                 trials=_log_int(rng, 1_000, 100_000), sum_mode=rng.choice(["f64", "kahan32"]))
        c["ylt"] = "f64" if c["sum_mode"] == "f64" else "f32"
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
@dataclass
class Table:
    elt_id: int
    event_ids: np.ndarray
    mean: np.ndarray
    sigma_i: np.ndarray
    sigma_c: np.ndarray
    max_loss: np.ndarray
    retention: float
    limit: float
    share: float


@dataclass
class Cover:
    elts: List[Table]
    occ_retention: float
    occ_limit: float
    agg_retention: float
    agg_limit: float
    program_id: int = 0


@dataclass
class Book:
    layers: List[Cover]
    seed: int
    su_enabled: bool
    keying: int

    @property
    def n_elts(self) -> int:
        return sum(len(l.elts) for l in self.layers)


@dataclass
class Years:
    offsets: np.ndarray
    n_catalogue: int


def _f32(x: float) -> float:
    return x if math.isinf(x) else float(np.float32(x))


def _rng(seed, *more):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), *more])))


def _table(rng, elt_id, case) -> Table:
    n = int(case["rows"])
    ev = np.sort(rng.choice(case["catalogue"], size=n, replace=False, shuffle=False))
    mean = np.exp(rng.normal(12.0, 1.5, size=n)).astype(np.float32)
    law = case["law"]
    si = mean * np.float32(0.25 if law == "mix" else 0.5)
    sc = si.copy() if law == "mix" else np.zeros(n, np.float32)
    mx = mean * np.float32(4.0)
    if law == "varied":
        si = (mean * rng.uniform(0.15, 0.9, n)).astype(np.float32)
        mx = (mean * rng.uniform(1.5, 10.0, n)).astype(np.float32)
    elif law == "capped":
        si = np.where(rng.random(n) < 0.3, np.float32(3.0) * mean, si).astype(np.float32)
    s = case["scale"]
    return Table(elt_id, ev.astype(np.int32), mean, si, sc, mx, _f32(LIMITS["elt_r"] * s),
                 _f32(LIMITS["elt_l"] * s), 1.0)


def _book(case, seed, index=0) -> Book:
    rng = _rng(seed, 1, index)
    layers, eid = [], 1000 * index
    for l in range(int(case["layers"])):
        s = case["scale"]
        t = [_f32(LIMITS[k] * s) for k in ("occ_r", "occ_l", "agg_r", "agg_l")]
        if case.get("fit"):
            # a drawn book's layer terms follow its size, so that it pays in some years
            hits = case["elts"] * case["rows"] / case["catalogue"]
            few = 1.0 if case["su"] else 0.1       # means alone seldom reach the retentions
            occ, agg = min(1.0, hits / 3.2), min(1.0, hits * case["lam"] / 3200.0)
            v = np.exp(rng.uniform(math.log(0.1), 0.0, size=2))
            t = [_f32(t[0] * few * occ * float(v[0])), t[1],
                 _f32(t[2] * few * agg * float(v[1])), _f32(LIMITS["agg_l"] * 4.0 * agg)]
        elif case.get("terms", "random") == "random":
            # retentions and limits of a programme's layers lie decades apart
            v = np.exp(rng.uniform(math.log(1e5), math.log(1e9), size=4)) * s
            t = [_f32(float(x)) for x in v]
        elts = []
        for _ in range(int(case["elts"])):
            elts.append(_table(rng, eid, case))
            eid += 1
        layers.append(Cover(elts, *t, program_id=l % 3))
    return Book(layers, seed=(int(seed) * 7919 + 13 * index + 5) & 0xFFFFFFFFFFFF,
                su_enabled=bool(case["su"]), keying=int(case.get("keying", 0)))


def _years(case, seed):
    """Poisson occurrences per year (given their sum, so that every seed has as
    many occurrences), events uniform over the catalogue."""
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(int(seed) * 2 + 1)
    n = int(case["trials"])
    lam = torch.full((n,), float(case["lam"]), dtype=torch.float32, device=dev)
    off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    counts = torch.poisson(lam, generator=g).to(torch.int64)
    short = int(n * case["lam"]) - int(counts.sum())
    years = torch.randint(0, n, (abs(short),), device=dev, generator=g)
    counts.index_add_(0, years, torch.full_like(years, 1 if short > 0 else -1))
    torch.cumsum(counts.clamp_(min=0), 0, out=off[1:])
    off.clamp_(max=int(n * case["lam"]))
    off[n] = int(n * case["lam"])
    host = off.cpu().numpy()
    ev = torch.randint(0, int(case["catalogue"]), (int(host[-1]),), dtype=torch.int32, device=dev,
                       generator=g)
    return off, ev, host


def _ylt(case, seed):
    """Yearly losses as a layer gives them: many zeros, a long tail, ties at the limit."""
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(int(seed) * 2 + 1)
    dt = torch.float64 if case["ylt"] == "f64" else torch.float32
    y = torch.randn(int(case["trials"]), dtype=torch.float64, device=dev, generator=g)
    return (torch.exp(17.0 + 1.5 * y) - 2e7).clamp(0.0, 1e9).to(dt)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
_CONTEXT = None


def _context():
    global _CONTEXT
    if _CONTEXT is None:
        from paper_1501_06326_amd import Ara
        _CONTEXT = Ara(0)
    return _CONTEXT


class State:
    """What a caller holds: the context's YET and portfolio handles."""

    def __init__(self, case):
        self.case = case
        self.ara = _context()
        self.yet = None
        self.loaded = []
        self.book = None
        self.ylt = None

    def __del__(self):
        try:
            for p in self.loaded:
                self.ara.free_portfolio(p)
            if self.yet is not None:
                self.ara.free_yet(self.yet)
        except Exception:
            pass


def prepare(case, seed):
    st = State(case)
    if case["kind"] == "metrics":
        st.ylt = _ylt(case, seed)
        return st
    off, ev, host = _years(case, seed)
    st.yet = st.ara.load_yet(Years(host, int(case["catalogue"])), device_arrays=(off, ev, None))
    if case["kind"] == "price":
        st.book = _book(case, seed)
        return st
    for i in range(int(case.get("portfolios", 1))):
        st.loaded.append(st.ara.load_portfolio(_book(case, seed, i), int(case["catalogue"])))
    return st


def run(st):
    case, ara = st.case, st.ara
    if case["kind"] == "metrics":
        pml, tvar = ara.pml_tvar(st.ylt, RETURN_PERIODS[:int(case["periods"])])
        srt, mean = ara.ep_curve(st.ylt)
        return {"pml": pml, "tvar": tvar, "sorted": srt, "tail_mean": mean}
    if case["kind"] == "batch":
        return ara.run_batch(st.yet, st.loaded, sum_mode=case["sum_mode"],
                             ylt_dtype=case["ylt"], sync=False)
    if case["kind"] == "price":
        p = ara.load_portfolio(st.book, int(case["catalogue"]))
        out = ara.run(st.yet, p, sum_mode=case["sum_mode"], ylt_dtype=case["ylt"])
        ara.free_portfolio(p)
        return out
    return ara.run(st.yet, st.loaded[0], sum_mode=case["sum_mode"], ylt_dtype=case["ylt"],
                   occ_view=bool(case["view"]), sync=False)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Bytes: event ids, offsets, the rows of the tables once, the outputs.
    Operations, with secondary uncertainty: per draw that can pay, 57 of the
    Philox rounds and 20 of a quantile read from a table; without: one
    addition per occurrence and layer."""
    n = float(case["trials"])
    size = 8.0 if case["ylt"] == "f64" else 4.0
    if case["kind"] == "metrics":
        return {"bytes": n * (2 * size + size + 8.0), "flops": n * 2.0}
    occ = n * case["lam"]
    pfs = float(case.get("portfolios", 1))
    layers = pfs * case["layers"]
    rows = layers * case["elts"] * case["rows"]
    out = n * size * (layers + pfs)
    if case.get("view"):
        out += occ * size * layers
    b = 4.0 * occ + 8.0 * n + 20.0 * rows + out
    if not case["su"]:
        return {"bytes": b, "flops": occ * layers}
    # a row pays where 4 x its lognormal mean exceeds the retention
    cut = (math.log(LIMITS["elt_r"] * case["scale"] / 4.0) - 12.0) / 1.5
    pay = 0.5 * math.erfc(cut / math.sqrt(2.0))
    draws = occ * layers * case["elts"] * (case["rows"] / case["catalogue"]) * pay
    return {"bytes": b, "flops": draws * (134.0 if case["law"] == "mix" else 77.0)}


# --------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Word 0 of Philox4x32-10 (Salmon et al., SC'11) on int64 tensors."""
    k0, k1 = int(seed) & _M32, (int(seed) >> 32) & _M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32,
                          ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0


def _grid(word):
    """The draw on the 2^-24 grid: u = j 2^-24, j odd."""
    return (word >> 8) | 1


def _fraction(a, b, x):
    """1 / K of I_x(a, b) = x^a (1-x)^b / (a B(a, b)) / K (DLMF 8.17.22), by the
    modified Lentz recurrence until no element moves."""
    tiny = 1e-300
    c = torch.ones_like(x)
    d = 1.0 - (a + b) * x / (a + 1.0)
    d = 1.0 / torch.where(d.abs() < tiny, tiny, d)
    h = d.clone()
    for m in range(1, 2000):
        for odd in (0, 1):
            if odd:
                t = -(a + m) * (a + b + m) * x / ((a + 2 * m) * (a + 2 * m + 1.0))
            else:
                t = m * (b - m) * x / ((a + 2 * m - 1.0) * (a + 2 * m))
            d = 1.0 + t * d
            d = 1.0 / torch.where(d.abs() < tiny, tiny, d)
            c = 1.0 + t / c
            c = torch.where(c.abs() < tiny, tiny, c)
            step = c * d
            h = h * step
        if m % 6 == 0 and float((step - 1.0).abs().max()) < 1e-15:
            break
    return h


def _beta_inc(a, b, lnb, x):
    """I_x, 1 - I_x and x f(x) for the density f."""
    e = torch.exp(a * torch.log(x) + b * torch.log1p(-x) - lnb)
    direct = x * (a + b + 2.0) < a + 1.0
    A, B = torch.where(direct, a, b), torch.where(direct, b, a)
    v = e * _fraction(A, B, torch.where(direct, x, 1.0 - x)) / A
    return torch.where(direct, v, 1.0 - v), torch.where(direct, 1.0 - v, v), e / (1.0 - x)


def _beta_quantile(a, b, z, zc):
    """x with I_x(a, b) = z, given zc = 1 - z as well: safeguarded Newton steps
    on the logarithms, on the side of the root that is at most one half."""
    lnb = torch.lgamma(a) + torch.lgamma(b) - torch.lgamma(a + b)
    ih, ihc, _ = _beta_inc(a, b, lnb, torch.full_like(a, 0.5))
    low = torch.where(z <= zc, z <= ih, zc >= ihc)
    A, B = torch.where(low, a, b), torch.where(low, b, a)
    Z, ZC = torch.where(low, z, zc), torch.where(low, zc, z)
    y0 = (torch.log(Z) + torch.log(A) + lnb) / A
    res = torch.zeros_like(a)
    live = torch.nonzero(y0 > -690.0).flatten()      # below, the root is 0 to any precision
    A, B, Z, ZC, ln = A[live], B[live], Z[live], ZC[live], lnb[live]
    hi = torch.full_like(A, math.log(0.5))
    lo = torch.full_like(A, -700.0)
    y = torch.minimum(y0[live], hi - 0.05)
    small = Z <= ZC
    for _ in range(80):
        i, ic, xf = _beta_inc(A, B, ln, torch.exp(y))
        f = torch.where(small, torch.log(i) - torch.log(Z), torch.log(ZC) - torch.log(ic))
        slope = xf / torch.where(small, i, ic)
        hi, lo = torch.where(f > 0, y, hi), torch.where(f > 0, lo, y)
        step = f / slope
        yn = y - step
        still = step.abs() <= 1e-14 * (1.0 + y.abs())
        out = ~((yn > lo) & (yn < hi) & torch.isfinite(yn)) & ~still
        yn = torch.where(out, 0.5 * (lo + hi), yn)
        moved = ~still
        y = yn
        if not bool(moved.any()):
            break
        if float(moved.float().mean()) < 0.5:        # go on with those that still move
            res[live] = torch.exp(y)
            keep = torch.nonzero(moved).flatten()
            live, A, B, Z, ZC, ln = (t[keep] for t in (live, A, B, Z, ZC, ln))
            hi, lo, y, small = hi[keep], lo[keep], y[keep], small[keep]
    if live.numel():
        res[live] = torch.exp(y)
    return torch.where(low, res, 1.0 - res)


def _shapes(t: Table):
    """Beta moment fit of a table's rows: a, b, with the cap at the largest
    standard deviation."""
    mu, mx = t.mean.astype(np.float64), t.max_loss.astype(np.float64)
    sg = t.sigma_i.astype(np.float64) + t.sigma_c.astype(np.float64)
    mb = mu / mx
    top = np.sqrt(mb * (1.0 - mb))
    sb = np.where(sg / mx >= top, (1.0 - 1e-6) * top, sg / mx)
    kappa = (top / sb) ** 2 - 1.0
    return mb * kappa, (1.0 - mb) * kappa


class _Rows:
    """One table on the device: its paying rows' columns and, by event, 1 + row."""

    def __init__(self, t: Table, case, dev):
        f = lambda v: torch.from_numpy(np.ascontiguousarray(v, np.float64)).to(dev)  # noqa: E731
        scale = t.max_loss if case["su"] else t.mean
        pays = scale > np.float32(t.retention)
        self.t = t
        idx = np.zeros(case["catalogue"], np.int32)
        idx[t.event_ids[pays]] = np.arange(1, int(pays.sum()) + 1, dtype=np.int32)
        self.of_event = torch.from_numpy(idx).to(dev)
        self.mean, self.top = f(t.mean[pays]), f(t.max_loss[pays])
        if case["su"]:
            a, b = _shapes(t)
            self.a, self.b = f(a[pays]), f(b[pays])
            si, sc = t.sigma_i[pays].astype(np.float64), t.sigma_c[pays].astype(np.float64)
            self.wc = f(sc / (si + sc))


def _single_table(a, b, dev):
    """The quantile of one shape at every point of the draw grid."""
    x = torch.empty(1 << 23, dtype=torch.float64, device=dev)
    for c in range(0, 1 << 23, 1 << 21):
        j = (2 * torch.arange(c, c + (1 << 21), device=dev) + 1).to(torch.float64)
        z = j / 16777216.0
        x[c:c + (1 << 21)] = _beta_quantile(torch.full_like(z, a), torch.full_like(z, b), z,
                                            (16777216.0 - j) / 16777216.0)
    return x


def _layer_losses(case, book, cover, rows, tables, ev, k, trial):
    """Loss of each occurrence net of the layer's occurrence terms."""
    X = torch.zeros(ev.numel(), dtype=torch.float64, device=ev.device)
    e64 = ev.to(torch.int64)
    for R in rows:
        t = R.t
        r = R.of_event[e64]
        at = torch.nonzero(r).flatten()
        if at.numel() == 0:
            continue
        r = (r[at] - 1).to(torch.int64)
        if not case["su"]:
            loss = R.mean[r]
        else:
            kk, ii = k[at], trial[at]
            zero = torch.zeros_like(kk)
            if book.keying:
                w = _philox(kk, ii, zero + cover.program_id, zero + 2, book.seed)
            else:
                w = _philox(kk, ii, zero + t.elt_id, zero, book.seed)
            jI = _grid(w)
            if case["law"] == "mix":
                if book.keying:
                    w = _philox(e64[at], zero, zero, zero + 3, book.seed)
                else:
                    w = _philox(kk, ii, zero, zero + 1, book.seed)
                jC = _grid(w)
                s = 1.0 / 16777216.0
                wc = R.wc[r]
                wi = 1.0 - wc
                nI = torch.special.ndtri(jI.to(torch.float64) * s)
                nC = torch.special.ndtri(jC.to(torch.float64) * s)
                v = (nI * wi + nC * wc) / torch.sqrt(wi * wi + wc * wc)
                q = math.sqrt(0.5)
                z, zc = 0.5 * torch.special.erfc(-v * q), 0.5 * torch.special.erfc(v * q)
                x = _beta_quantile(R.a[r], R.b[r], z, zc)
            elif tables is not None:
                x = tables[jI >> 1]
            else:
                j = jI.to(torch.float64)
                x = _beta_quantile(R.a[r], R.b[r], j / 16777216.0, (16777216.0 - j) / 16777216.0)
            loss = R.top[r] * x
        X.index_add_(0, at, t.share * (loss - t.retention).clamp(0.0, t.limit))
    return (X - cover.occ_retention).clamp(0.0, cover.occ_limit)


def _exact_run(case, book, off, ev, host):
    dev = ev.device
    n = int(case["trials"])
    ylt = torch.zeros((len(book.layers), n), dtype=torch.float64, device=dev)
    view = (torch.zeros((len(book.layers), max(1, ev.numel())), dtype=torch.float64, device=dev)
            if case.get("view") else None)
    single = case["su"] and case["law"] == "single"
    tables = _single_table(0.25 * 11.0, 0.75 * 11.0, dev) if single else None
    per = max(1, int((20e6 if single or not case["su"] else 4e6) / max(1.0, case["lam"])))
    for l, cover in enumerate(book.layers):
        rows = [_Rows(t, case, dev) for t in cover.elts]
        for t0 in range(0, n, per):
            t1 = min(n, t0 + per)
            a, b = int(host[t0]), int(host[t1])
            counts = off[t0 + 1:t1 + 1] - off[t0:t1]
            trial = torch.repeat_interleave(torch.arange(t0, t1, device=dev), counts)
            start = torch.repeat_interleave(off[t0:t1], counts)
            k = torch.arange(a, b, device=dev) - start
            O = _layer_losses(case, book, cover, rows, tables, ev[a:b], k, trial)
            total = torch.zeros(t1 - t0, dtype=torch.float64, device=dev)
            total.index_add_(0, trial - t0, O)
            ylt[l, t0:t1] = (total - cover.agg_retention).clamp(0.0, cover.agg_limit)
            if view is not None and b > a:
                S = torch.cumsum(O, 0)
                before = torch.cat([S.new_zeros(1), S])[start - a]
                A = (S - before - cover.agg_retention).clamp(0.0, cover.agg_limit)
                prev = torch.cat([A.new_zeros(1), A[:-1]])
                view[l, a:b] = A - torch.where(k == 0, 0.0, prev)
    out = {"ylt": ylt, "ylt_pf": ylt.sum(0)}
    if view is not None:
        out["occ_view"] = view
    return out


def _exact_cost(case):
    """Rough seconds of ``exact``."""
    draws = work(case)["flops"] / 77.0 if case.get("su") else 0.0
    walk = case["trials"] * case["lam"] * case["layers"] * case["elts"] * case.get("portfolios", 1)
    per = {"single": 4e-9, "mix": 6e-8, "varied": 2.5e-7, "capped": 1.5e-7}[case["law"]]
    return draws * per + walk * 2.0e-10


def exact(case, seed):
    if case["kind"] == "metrics":
        y = _ylt(case, seed).to(torch.float64)
        srt = torch.sort(y, descending=True).values
        mean = torch.cumsum(srt, 0) / torch.arange(1, y.numel() + 1, device=y.device)
        n = y.numel()
        periods = RETURN_PERIODS[:int(case["periods"])]
        ks = [max(1, min(n, int(math.floor(n / rp)))) for rp in periods]
        return {"pml": np.array([float(srt[k - 1]) for k in ks]),
                "tvar": np.array([float(mean[k - 1]) for k in ks]), "sorted": srt,
                "tail_mean": mean}
    if _exact_cost(case) > 15.0:
        return None
    off, ev, host = _years(case, seed)
    if case["kind"] == "batch":
        return [_exact_run(case, _book(case, seed, i), off, ev, host)
                for i in range(int(case["portfolios"]))]
    return _exact_run(case, _book(case, seed), off, ev, host)
