"""The occurrence view without secondary uncertainty over short years.

A year that fits one aligned group of four ids a lane is scanned in one piece: every
length around its edges at every alignment of the ids, where the tables are read from
each place.  The Year Loss Table is that of the run without a view, bit for bit; the
view is the oracle's within the 2 (1e-5 G + 1e-3) of its other tests, and each year's
increments add up to its loss within 1e-5 G + 1e-3.
"""
import numpy as np
import pytest

import oracle
from workloads import ELT, YET, Layer, Portfolio

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


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("n_cat,n,what", [(1000, 34_000, "dense"), (30_011, 34_000, "sparse"),
                                          (1_000_000, 34_000, "bitmap"), (3_000_000, 4_000, "global")])
def test_short_years(ara, n_cat, n, what, shift):
    rng = np.random.default_rng(n_cat + shift)
    rows = min(n_cat // 2, 9000)
    ev = np.sort(rng.choice(n_cat, rows, replace=False)).astype(np.int32)
    m = np.exp(rng.normal(12, 1, rows)).astype(np.float32) + np.float32(2000.0)
    zero = np.zeros(rows, np.float32)
    elt = ELT(elt_id=1, event_ids=ev, mean=m, sigma_i=zero, sigma_c=zero, max_loss=2 * m,
              retention=1e3, limit=1e9, share=0.9)
    pf = Portfolio(layers=[Layer(elts=[elt], occ_retention=1e4, occ_limit=1e7, agg_retention=1e5,
                                 agg_limit=1e8)], seed=5, su_enabled=False)
    lens = rng.integers(0, 264, n)
    lens[:24] = [0, 1, 2, 3, 4, 5, 6, 7, 8, 60, 61, 62, 63, 64, 65, 249, 250, 251, 252, 253, 254, 255, 256, 257]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    assert what != "bitmap" or off[-1] >= 4_100_000
    ids = rng.integers(0, n_cat, off[-1]).astype(np.int32)
    hit = rng.random(off[-1]) < 0.5
    ids[hit] = rng.choice(ev, int(hit.sum()))
    yet = YET(offsets=off, event_ids=ids, times=None, n_catalogue=n_cat)
    # the ids begin shift elements behind an aligned address
    buf = torch.zeros(off[-1] + shift, dtype=torch.int32, device="cuda")
    buf[shift:] = torch.from_numpy(ids).cuda()
    d_off = torch.from_numpy(off).cuda()
    y = ara.load_yet(yet, device_arrays=(d_off, buf[shift:], None))
    p = ara.load_portfolio(pf, n_cat)
    print("short years", what, shift, flush=True)
    few = 300
    ref = oracle.run_ara(YET(offsets=off[:few + 1], event_ids=ids[:off[few]], times=None,
                             n_catalogue=n_cat), pf, occ_view=True)
    G = ref["gross"][0]
    for mode, dtype in (("kahan32", "f32"), ("naive32", "f32"), ("f64", "f64")):
        r = ara.run(y, p, sum_mode=mode, ylt_dtype=dtype)
        v = ara.run(y, p, sum_mode=mode, ylt_dtype=dtype, occ_view=True)
        assert torch.equal(r["ylt"], v["ylt"]) and torch.equal(r["ylt_pf"], v["ylt_pf"])
        d = v["occ_view"][0].double().cpu().numpy()
        assert d.size == off[-1]
        tol = 1e-5 * G + 1e-3
        assert np.all(np.abs(d[:off[few]] - ref["occ_view"][0]) <= 2 * np.repeat(tol, lens[:few]))
        total = np.concatenate([[0.0], np.cumsum(d)])[off]
        Y = r["ylt"][0].double().cpu().numpy()
        assert np.all(np.abs(np.diff(total)[:few] - Y[:few]) <= tol)
        s = ara.run(y, p, trial_begin=100, trial_count=150, sum_mode=mode, ylt_dtype=dtype, occ_view=True)
        assert torch.equal(s["occ_view"][0], v["occ_view"][0, off[100]:off[250]])
    ara.free_portfolio(p)
    ara.free_yet(y)
