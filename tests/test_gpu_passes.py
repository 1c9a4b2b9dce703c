"""The passes of a run with secondary uncertainty give the same trial the same bits.

The pass is chosen by the size of the run and by its rows (``debug_run_pass``), so a
run, its slices, its diagnostic pass and a batch may each take another one."""
import numpy as np
import pytest

import oracle
from test_gpu_segments import table_case
from workloads import YET, Layer, Portfolio, make_elt

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


# Events of up to 12 rows (whole chunks of 64 occurrences) and of 13, 14 and 15, whose
# segments end between multiples of 64; the event filter with such; a layer of more ELTs
# than are staged in LDS; small catalogues, one to four layers.
@pytest.mark.parametrize("sum_mode,dtype", [("naive32", "f32"), ("f64", "f64"), ("kahan32", "f32")])
@pytest.mark.parametrize("n_cat,n_elts,rows,layers", [
    (4096, 12, 4000, 2), (4096, 13, 3900, 2), (4097, 14, 4097, 3), (4096, 15, 3900, 1),
    (33, 3, 20, 4), (128_513, 13, 100_000, 2), (9_999, 70, 300, 4)])
def test_table_form_sums_like_the_others(ara, n_cat, n_elts, rows, layers, sum_mode, dtype):
    from paper_1501_06326_amd.ara import ARA_PASS_LEAN, ARA_PASS_TABLE
    n = 16_384
    # one layer of more rows than events takes the form where its ids outgrow the last-level cache
    lam = 800 if layers > 1 else 4200
    yet, pf = table_case(n_cat, n_elts, rows, n, lam, layers)
    print("table form sums", n_cat, n_elts, rows, layers, sum_mode, flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    how = dict(sum_mode=sum_mode, ylt_dtype=dtype)
    assert ara.debug_run_pass(y, p) == ARA_PASS_TABLE
    r = ara.run(y, p, **how)
    assert float(r["ylt"].max()) > 0
    for a, b in ((0, 2000), (n - 2000, n)):
        assert ara.debug_run_pass(y, p, trial_begin=a, trial_count=b - a) == ARA_PASS_LEAN
        for diag in (False, True):
            s = ara.run(y, p, trial_begin=a, trial_count=b - a, diagnostics=diag, **how)
            assert torch.equal(r["ylt"][:, a:b], s["ylt"])
            assert torch.equal(r["ylt_pf"][a:b], s["ylt_pf"])
    assert all(torch.equal(q["ylt"], r["ylt"]) for q in ara.run_batch(y, [p, p], **how))
    v = ara.run(y, p, occ_view=True, **how)
    assert torch.equal(v["ylt"], r["ylt"])
    s = ara.run(y, p, trial_count=2000, occ_view=True, **how)
    assert torch.equal(v["occ_view"][:, :s["occ_view"].shape[1]], s["occ_view"])
    ara.free_portfolio(p)
    ara.free_yet(y)


def odd_rows_case(n_iter, n_f64, n_mix, keying, layers=1):
    """6,000 years of 60 occurrences on average over 2,000 events; one shape but for
    n_iter rows of their own shape in [1, 32], n_f64 of FP64 shapes and n_mix mixed ones
    of their own shape, which all pay."""
    rng = np.random.default_rng(17)
    n_cat, n = 2000, 6000
    counts = rng.poisson(60.0, n)
    counts[:3] = [0, 1, 700]
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(counts)
    yet = YET(offsets=off, event_ids=rng.integers(0, n_cat, off[-1]).astype(np.int32), times=None,
              n_catalogue=n_cat)
    ls = []
    for l in range(layers):
        elts = [make_elt(10 * l + e, 700, n_cat, 5 * l + e, retention=1e3, limit=5e7) for e in range(5)]
        e, at = elts[2], rng.permutation(700)[:n_iter + n_f64 + n_mix]
        e.mean[at] = np.maximum(e.mean[at], np.float32(1e5))
        e.max_loss[at] = 4 * e.mean[at]
        a, b, c = np.split(at, [n_iter, n_iter + n_f64])
        e.sigma_i[a] = e.mean[a] * (0.4 + 0.2 * rng.random(a.size)).astype(np.float32)
        e.sigma_i[b] = e.mean[b] * (1.1 + 3.0 * rng.random(b.size)).astype(np.float32)
        e.sigma_i[c] = e.mean[c] * (0.2 + 0.1 * rng.random(c.size)).astype(np.float32)
        e.sigma_c[c] = e.sigma_i[c]
        ls.append(Layer(elts=elts, occ_retention=1e4, occ_limit=2e8, agg_retention=1e5, agg_limit=1e12,
                        program_id=l))
    return yet, Portfolio(layers=ls, seed=8, keying=keying)


# Rows without a slot: by the FP32 iteration in the lean pass, handed over, or by the
# full pass alone; 60 occurrences over 2,000 events make a hit on one of 5 rows in one
# trial of seven, on one of 400 in all of them.  (The first 16 shapes have slots, those of
# mixed rows too.)
@pytest.mark.parametrize("n_iter,n_f64,n_mix,keying,layers,want", [
    (0, 0, 0, 0, 1, 0), (20, 0, 0, 0, 1, 3), (400, 0, 0, 1, 1, 3), (0, 5, 0, 0, 1, 0),
    (30, 3, 2, 0, 2, 3), (40, 0, 4, 1, 1, 3), (0, 400, 0, 0, 1, 2), (200, 200, 200, 0, 2, 2)])
def test_odd_rows(ara, n_iter, n_f64, n_mix, keying, layers, want):
    """The pass that the rows ask for; the oracle within the 1e-5 G + 1e-3 of the other
    parity tests; a slice whose trials are all resident (there the full pass runs alone
    when one of them has an FP64 hit), the diagnostic pass, the view and batches in both
    orders bit for bit."""
    from paper_1501_06326_amd.ara import ARA_PASS_FULL
    yet, pf = odd_rows_case(n_iter, n_f64, n_mix, keying, layers)
    print("odd rows", n_iter, n_f64, n_mix, keying, flush=True)
    ref = oracle.run_ara(yet, pf)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, yet.n_catalogue)
    assert ara.debug_run_pass(y, p) == want
    assert ara.debug_run_pass(y, p, diagnostics=True) == want
    r = ara.run(y, p)
    err = np.abs(r["ylt"].double().cpu().numpy() - ref["ylt"])
    assert np.all(err <= 1e-5 * ref["gross"] + 1e-3)
    if n_f64 + n_mix:
        assert ara.debug_run_pass(y, p, trial_count=3000) == ARA_PASS_FULL
    s = ara.run(y, p, trial_begin=100, trial_count=3000)
    assert torch.equal(s["ylt"], r["ylt"][:, 100:3100])
    d = ara.run(y, p, diagnostics=True)
    assert torch.equal(d["ylt"], r["ylt"])
    assert np.array_equal(d["hits"].cpu().numpy(), ref["hits"])
    assert np.array_equal(d["hit_chk"].cpu().numpy().astype(np.uint64), ref["hit_chk"])
    v = ara.run(y, p, occ_view=True)
    assert torch.equal(v["ylt"], r["ylt"])
    s = ara.run(y, p, trial_count=3000, occ_view=True)
    assert torch.equal(v["occ_view"][:, :s["occ_view"].shape[1]], s["occ_view"])
    for band in (1e-4, 0.01):
        w = ara.run(y, p, tail_band=band)
        q = ara.run(y, p, trial_begin=100, trial_count=3000, tail_band=band)
        assert torch.equal(q["ylt"], w["ylt"][:, 100:3100])
    yet2, pf2 = odd_rows_case(30, 5, 0, 0)
    p2 = ara.load_portfolio(pf2, yet.n_catalogue)
    for cfg in (None, (2, 4, 1), (1, 0, 1)):
        o = ara.run_batch(y, [p, p2, p], cfg=cfg)
        assert torch.equal(o[0]["ylt"], r["ylt"]) and torch.equal(o[2]["ylt_pf"], r["ylt_pf"])
        assert torch.equal(o[1]["ylt"], ara.run(y, p2)["ylt"])
    for h in (p, p2):
        ara.free_portfolio(h)
    ara.free_yet(y)


def test_mixed_rows_all_resident(ara):
    """10.8 million mixed draws in 4,000 resident trials: more than one is expected beyond
    2^-24, so the full pass runs alone; slices, where none is, take the lean pass and give
    the same bits."""
    from paper_1501_06326_amd.ara import ARA_PASS_FULL, ARA_PASS_LEAN
    rng = np.random.default_rng(2)
    n_cat, n = 500, 4000
    off = np.arange(n + 1, dtype=np.int64) * 600
    yet = YET(offsets=off, event_ids=rng.integers(0, n_cat, off[-1]).astype(np.int32), times=None,
              n_catalogue=n_cat)
    pf = Portfolio(layers=[Layer(elts=[make_elt(e, 450, n_cat, e, corr=True, retention=1e3, limit=5e7)
                                       for e in range(5)], occ_retention=1e4, occ_limit=2e8,
                                 agg_retention=1e5, agg_limit=1e12)], seed=3)
    print("mixed rows, all resident", flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    assert ara.debug_run_pass(y, p) == ARA_PASS_FULL
    r = ara.run(y, p)
    for a in range(0, n, 1000):
        assert ara.debug_run_pass(y, p, trial_begin=a, trial_count=1000) == ARA_PASS_LEAN
        s = ara.run(y, p, trial_begin=a, trial_count=1000)
        assert torch.equal(s["ylt"], r["ylt"][:, a:a + 1000])
    ara.free_portfolio(p)
    ara.free_yet(y)


@pytest.mark.parametrize("n_elts,rows,layers,n,lam,want", [
    (6, 3000, 4, 9000, 280, 0), (12, 12_000, 2, 5000, 1500, 0), (12, 12_000, 2, 8192, 1500, 1)])
def test_layers_beyond_the_cache(ara, n_elts, rows, layers, n, lam, want):
    """Runs whose layers' tables exceed a cache: with fewer wavefronts a CU, and at the
    line of the event-table form (5,000 trials fill its second round to a fifth), the bits
    of a slice, of the diagnostic pass and of a batch in both orders."""
    n_cat = 250_007
    yet, pf = table_case(n_cat, n_elts, rows, n, lam, layers)
    print("layers beyond the cache", layers, n, flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    assert ara.debug_run_pass(y, p) == want
    r = ara.run(y, p)
    assert float(r["ylt"].max()) > 0
    s = ara.run(y, p, trial_begin=n - 2000, trial_count=2000)
    assert torch.equal(s["ylt"], r["ylt"][:, n - 2000:])
    d = ara.run(y, p, diagnostics=True)
    assert torch.equal(d["ylt"], r["ylt"]) and torch.equal(d["ylt_pf"], r["ylt_pf"])
    v = ara.run(y, p, occ_view=True)
    assert torch.equal(v["ylt"], r["ylt"])
    for cfg in (None, (1, 0, 1)):
        o = ara.run_batch(y, [p, p], cfg=cfg)
        assert all(torch.equal(q["ylt"], r["ylt"]) for q in o)
    ara.free_portfolio(p)
    ara.free_yet(y)
