"""Quantiles of secondary uncertainty at their edges: polynomial segments, the FP64
path, and the queues of the full pass.

The quantile of shapes with a slot, at the edges of its polynomial segments.

By draw: grid points on both sides of every octave edge of min(z, 1 - z), both
halves, against the FP64 oracle's inverse.  Bound: the segments interpolate to
below 2e-7 of the root (degree 7 over an octave; the worst shape of [1, 32]^2 is
(1, 32)), the FP32 coefficients and the last Horner step round to 1.2e-7
together, so 4e-7 of max(root, mean).

By normal deviate: portfolios of the two-normal mix with unequal parts, against
the oracle's run, with the per-trial bound 1e-5 G + 1e-3 of the other parity tests.
"""
import numpy as np
import pytest

import oracle
from workloads import config_small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ara():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06326_amd import Ara
    a = Ara(0)
    yield a
    a.close()


@pytest.mark.parametrize("a,b", [(2.75, 8.25), (1.0, 1.0), (1.0, 32.0), (32.0, 1.0), (32.0, 32.0)])
def test_octave_edges(ara, a, b):
    edges = 2 ** np.arange(1, 24, dtype=np.int64)
    j = np.concatenate([[1], edges - 1, edges[:-1] + 1, edges[2:] - 3])
    j = np.unique(np.concatenate([j, (1 << 24) - j]))
    assert np.all(j % 2 == 1) and j.min() == 1 and j.max() == (1 << 24) - 1
    z, zc = j / 2.0 ** 24, ((1 << 24) - j) / 2.0 ** 24
    print("octave edges", a, b, flush=True)
    x, path = ara.debug_beta_quantile_shape(a, b, z, zc)
    ref = oracle.betaincinv(a, b, z, zc)
    assert np.all(path == 0)
    assert np.max(np.abs(x - ref) / np.maximum(ref, a / (a + b))) <= 4e-7


@pytest.mark.parametrize("part", [0.02, 0.3, 0.95])
def test_mixed_rows_unequal_parts(ara, part):
    """sigma_C / sigma = part; one shape per ELT, so every row has a slot."""
    w = config_small(n_trials=1500)
    for e in w.portfolio.layers[0].elts:
        e.sigma_c = (e.sigma_i * np.float32(part)).astype(np.float32)
        e.sigma_i = (e.sigma_i * np.float32(1.0 - part)).astype(np.float32)
    print("mixed rows", part, flush=True)
    ref = oracle.run_ara(w.yet, w.portfolio)
    y = ara.load_yet(w.yet)
    p = ara.load_portfolio(w.portfolio, w.yet.n_catalogue)
    r = ara.run(y, p)
    err = np.abs(r["ylt"].double().cpu().numpy() - ref["ylt"])
    assert np.all(err <= 1e-5 * ref["gross"] + 1e-3)
    # a wide tail band hands draws to the FP64 quantile: the same trials within the bound
    r2 = ara.run(y, p, tail_band=0.01)
    assert np.all(np.abs(r2["ylt"].double().cpu().numpy() - ref["ylt"]) <= 1e-5 * ref["gross"] + 1e-3)
    ara.free_portfolio(p)
    ara.free_yet(y)


# FP64 quantile: shapes outside the FP32 domain.  It ends on a Halley step below
# 1e-4 of the root, whose error is the step's cube (1e-12) times a constant of
# order ten; the result is FP32, so 1e-7 of max(root, mean).
@pytest.mark.parametrize("a,b", [(0.3, 0.4), (0.02, 3.0), (5e-7, 1.5e-6), (0.7, 60.0), (40.0, 2.0),
                                 (33.0, 33.0), (400.0, 30.0), (5.0, 0.5), (2e4, 1e4)])
def test_fp64_quantile(ara, a, b):
    rng = np.random.default_rng(11)
    j = 2 * rng.integers(0, 1 << 23, 4000) + 1
    j[:8] = [1, 3, 5, (1 << 24) - 1, (1 << 24) - 3, (1 << 23) - 1, (1 << 23) + 1, 12345]
    z, zc = j / 2.0 ** 24, ((1 << 24) - j) / 2.0 ** 24
    print("fp64 quantile", a, b, flush=True)
    A, B = np.full(j.size, a, np.float32), np.full(j.size, b, np.float32)
    x, path = ara.debug_beta_quantile(A, B, z, zc)
    ref = oracle.betaincinv(float(A[0]), float(B[0]), z, zc)
    assert np.all(path == 1)
    assert np.max(np.abs(x - ref) / np.maximum(ref, a / (a + b))) <= 1e-7


@pytest.mark.parametrize("n_occ", [1, 63, 64, 65, 130, 511, 512, 513, 1100])
def test_full_pass_queues(ara, n_occ):
    """Trials of n_occ occurrences over rows of every kind (no draw, slotted,
    FP32 iteration, FP64 shape, near-Bernoulli, mixed with and without a slot),
    so both queues of the full pass fill and drain at every remainder: the
    oracle within 1e-5 G + 1e-3, the diagnostic pass and a batch bit for bit."""
    from workloads import ELT, YET, Layer, Portfolio
    rng = np.random.default_rng(n_occ)
    n_cat, n_trials = 40, 12
    elts = []
    for e in range(6):
        n = 30
        ev = np.sort(rng.choice(n_cat, n, replace=False)).astype(np.int32)
        m = np.exp(rng.normal(12, 1, n)).astype(np.float32)
        frac = rng.choice([0.0, 0.1, 0.5, 0.8, 3.0], n).astype(np.float32)
        top = rng.choice([1.5, 4.0, 9.0], n).astype(np.float32)
        corr = rng.choice([0.0, 0.0, 0.4, 1.0], n).astype(np.float32)
        elts.append(ELT(elt_id=7 * e, event_ids=ev, mean=m,
                        sigma_i=(m * frac * (1 - corr)).astype(np.float32),
                        sigma_c=(m * frac * corr).astype(np.float32),
                        max_loss=(m * top).astype(np.float32), retention=1e5, limit=5e6, share=0.9))
    pf = Portfolio(layers=[Layer(elts=elts, occ_retention=1e5, occ_limit=2e7, agg_retention=1e6,
                                 agg_limit=1e12)], seed=99)
    off = np.arange(n_trials + 1, dtype=np.int64) * n_occ
    yet = YET(offsets=off, event_ids=rng.integers(0, n_cat, off[-1]).astype(np.int32), times=None,
              n_catalogue=n_cat)
    print("full pass queues", n_occ, flush=True)
    ref = oracle.run_ara(yet, pf)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    r = ara.run(y, p)["ylt"]
    err = np.abs(r.double().cpu().numpy() - ref["ylt"])
    assert np.all(err <= 1e-5 * ref["gross"] + 1e-3)
    d = ara.run(y, p, diagnostics=True)
    assert torch.equal(d["ylt"], r)
    assert np.array_equal(d["hits"].cpu().numpy(), ref["hits"])
    for cfg in (None, (2, 4, 1)):
        assert torch.equal(ara.run_batch(y, [p, p], cfg=cfg)[1]["ylt"], r)
    ara.free_portfolio(p)
    ara.free_yet(y)


def table_case(n_cat, n_elts, rows, n_trials, lam, layers=1, seed=3, **kw):
    """A YET and a portfolio of slotted rows for the event-table form."""
    from workloads import YET, Layer, Portfolio, make_elt
    rng = np.random.default_rng(seed)
    counts = rng.poisson(lam, n_trials)
    counts[:4] = [0, 1, 511, 1537]
    off = np.zeros(n_trials + 1, np.int64)
    off[1:] = np.cumsum(counts)
    yet = YET(offsets=off, event_ids=rng.integers(0, n_cat, off[-1]).astype(np.int32), times=None,
              n_catalogue=n_cat)
    ls = [Layer(elts=[make_elt(100 * l + e, rows, n_cat, 77 + 10 * l + e, retention=1e5, limit=5e7)
                      for e in range(n_elts)], occ_retention=1e5 * (l + 1), occ_limit=2e8,
                agg_retention=1e6, agg_limit=1e12, program_id=l) for l in range(layers)]
    return yet, Portfolio(layers=ls, seed=5, **kw)


# catalogues at the edges of a 16-event group and of the largest table (8,032
# groups); tables sparse, of up to 15 rows an event (chunks of 51) and of more
# (no table form); one layer and several; both keyings; a tail band that abandons
# trials in single layers.
@pytest.mark.parametrize("n_cat,n_elts,rows,layers,keying,band", [
    (33, 3, 20, 1, 0, 0.0), (4096, 15, 3900, 1, 1, 0.0), (4097, 17, 4097, 1, 0, 0.0),
    (128_512, 2, 30_000, 2, 0, 0.0), (128_513, 2, 30_000, 2, 0, 0.0), (9_999, 6, 2_000, 4, 0, 1e-5)])
def test_table_form_equals_slices(ara, n_cat, n_elts, rows, layers, keying, band):
    """A run large enough for the event-table form gives the YLT and the
    occurrence view of the same trials run in slices too small for it, bit for
    bit, and a batch the same."""
    n = 65_536 // layers
    yet, pf = table_case(n_cat, n_elts, rows, n, 520, layers, keying=keying)
    print("table form", n_cat, n_elts, rows, layers, flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    r = ara.run(y, p, tail_band=band)
    for a, b in ((0, 4000), (n - 3000, n)):
        s = ara.run(y, p, trial_begin=a, trial_count=b - a, tail_band=band)
        assert torch.equal(r["ylt"][:, a:b], s["ylt"])
        assert torch.equal(r["ylt_pf"][a:b], s["ylt_pf"])
    assert float(r["ylt"].max()) > 0
    v = ara.run(y, p, occ_view=True, tail_band=band)
    assert torch.equal(v["ylt"], r["ylt"])
    s = ara.run(y, p, trial_count=4000, occ_view=True, tail_band=band)
    assert torch.equal(v["occ_view"][:, :s["occ_view"].shape[1]], s["occ_view"])
    if band == 0.0:
        o = ara.run_batch(y, [p, p])
        assert all(torch.equal(q["ylt"], r["ylt"]) and torch.equal(q["ylt_pf"], r["ylt_pf"]) for q in o)
    ara.free_portfolio(p)
    ara.free_yet(y)


# The same at sizes that the rule gives to the table form: the last catalogue of the
# table and the first of the filter, the last with a bit per event, the first with a
# bit for two, one with a bit for four, several layers, many rows an event.
@pytest.mark.parametrize("n_cat,n_elts,rows,layers,keying,band", [
    (128_512, 3, 30_000, 1, 0, 0.0), (128_513, 3, 30_000, 1, 0, 0.0), (771_072, 2, 30_000, 1, 0, 0.0),
    (771_073, 2, 30_000, 1, 0, 0.0), (2_000_003, 4, 30_000, 1, 1, 0.0), (250_007, 3, 20_000, 2, 0, 1e-5),
    (4_096, 15, 3_900, 2, 1, 0.0), (9_999, 6, 1_500, 1, 0, 1e-5)])
def test_large_runs_equal_slices(ara, n_cat, n_elts, rows, layers, keying, band):
    n = 16_384
    yet, pf = table_case(n_cat, n_elts, rows, n, 800, layers, keying=keying)
    for layer in pf.layers:                    # rows at both ends of the catalogue
        layer.elts[0].event_ids[0], layer.elts[0].event_ids[-1] = 0, n_cat - 1
    yet.event_ids[:4] = [0, n_cat - 1, n_cat - 1, 0]
    yet.event_ids[-2:] = [n_cat - 1, 0]
    print("large runs", n_cat, n_elts, rows, layers, flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    r = ara.run(y, p, tail_band=band)
    assert float(r["ylt"].max()) > 0
    for a, b in ((0, 4000), (7000, 11_000), (n - 4000, n)):
        s = ara.run(y, p, trial_begin=a, trial_count=b - a, tail_band=band)
        assert torch.equal(r["ylt"][:, a:b], s["ylt"])
        assert torch.equal(r["ylt_pf"][a:b], s["ylt_pf"])
    v = ara.run(y, p, occ_view=True, tail_band=band)
    assert torch.equal(v["ylt"], r["ylt"])
    s = ara.run(y, p, trial_count=4000, occ_view=True, tail_band=band)
    assert torch.equal(v["occ_view"][:, :s["occ_view"].shape[1]], s["occ_view"])
    if band == 0.0:
        o = ara.run_batch(y, [p, p])
        assert all(torch.equal(q["ylt"], r["ylt"]) and torch.equal(q["ylt_pf"], r["ylt_pf"]) for q in o)
    ara.free_portfolio(p)
    ara.free_yet(y)
