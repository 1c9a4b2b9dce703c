"""The load's per-event offsets and row places at the edges of its tiles.

Rows of every kind (no draw, slotted, FP64, mixed, never paying) land where the
diagnostic pass, which reads the event-major arrays, and the lean and full passes,
which read the compact records, both agree with the oracle: hit counts and checksums
exactly, losses within the 1e-5 G + 1e-3 of the other parity tests.
"""
import numpy as np
import pytest

import oracle

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


@pytest.mark.parametrize("su", [True, False])
@pytest.mark.parametrize("n_cat", [1, 254, 255, 256, 257, 511, 512, 1023, 70_000])
def test_load_tiles(ara, n_cat, su):
    from workloads import ELT, YET, Layer, Portfolio
    rng = np.random.default_rng(n_cat)
    layers, eid = [], 0
    for sizes in ([1.0, 0.4, 0.0], [], [0.0], [0.7] * 9):
        elts = []
        for frac in sizes:
            n = min(n_cat, 9000, int(round(frac * n_cat)))
            ev = np.sort(rng.choice(n_cat, n, replace=False)).astype(np.int32)
            if n == n_cat:                       # the last event of a full table pays
                ev[-1] = n_cat - 1
            m = np.exp(rng.normal(12, 1, n)).astype(np.float32)
            sig = rng.choice([0.0, 0.3, 0.6], n).astype(np.float32)
            corr = rng.choice([0.0, 0.4, 1.0], n).astype(np.float32)
            # a third of the rows cannot pay: their largest loss is below the retention
            top = np.where(rng.random(n) < 0.33, np.float32(1.2), np.float32(8.0))
            m = np.where(top < 2, np.minimum(m, 5e4), m).astype(np.float32)
            elts.append(ELT(elt_id=eid, event_ids=ev, mean=m, sigma_i=(m * sig * (1 - corr)).astype(np.float32),
                            sigma_c=(m * sig * corr).astype(np.float32),
                            max_loss=(m * top).astype(np.float32), retention=6e4, limit=1e7, share=0.8))
            eid += 1
        layers.append(Layer(elts=elts, occ_retention=1e4, occ_limit=1e8, agg_retention=1e4, agg_limit=1e12))
    pf = Portfolio(layers=layers, seed=7, su_enabled=su)
    off = np.arange(41, dtype=np.int64) * 37
    ids = rng.integers(0, n_cat, off[-1]).astype(np.int32)
    ids[:2] = [0, n_cat - 1]
    yet = YET(offsets=off, event_ids=ids, times=None, n_catalogue=n_cat)
    print("load tiles", n_cat, su, flush=True)
    ref = oracle.run_ara(yet, pf)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    r = ara.run(y, p)
    tol = 1e-5 * ref["gross"] + 1e-3
    assert np.all(np.abs(r["ylt"].double().cpu().numpy() - ref["ylt"]) <= tol)
    if su:
        d = ara.run(y, p, diagnostics=True)
        assert np.array_equal(d["hits"].cpu().numpy(), ref["hits"])
        assert np.array_equal(d["hit_chk"].cpu().numpy().astype(np.uint64), ref["hit_chk"])
        assert torch.equal(d["ylt"], r["ylt"])
    ara.free_portfolio(p)
    ara.free_yet(y)
