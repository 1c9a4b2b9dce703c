"""Where the pass without secondary uncertainty reads its tables from: the forms of the
dispatch at their edges, and layers taken together.

A form or a group changes where a loss is read, not the order it is added in, so every
one gives the same bits.  The oracle's bound is that of the other parity tests,
1e-5 G + 1e-3 of the trial's gross loss G.
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


def sparse_rows(n_cat, lds):
    """Non-zero events of a layer whose sparse table takes lds bytes."""
    return lds // 4 - 2 * ((n_cat + 31) // 32) - 1


ONE, TWO = 156 * 1024, 78 * 1024
CASES = [
    (8192, [900], "dense"), (8193, [900], "sparse"),
    (100_003, [sparse_rows(100_003, TWO)], "two blocks a CU"),
    (100_003, [sparse_rows(100_003, TWO) + 1], "one block"),
    (100_003, [sparse_rows(100_003, ONE)], "one block, full"),
    (100_003, [sparse_rows(100_003, ONE) + 1], "bitmap"),
    (1_277_952, [40_000], "bitmap, full"), (1_277_953, [40_000], "global"),
    (50_021, [5000, 1, 7000], "three together"),
    (50_021, [9000, 0, 7000, 3000, 50], "four together and one"),
    (50_021, [sparse_rows(50_021, TWO), sparse_rows(50_021, TWO), 10], "two together and one"),
    (50_021, [sparse_rows(50_021, TWO), sparse_rows(50_021, TWO) + 1, 10], "one and two"),
]


@pytest.mark.parametrize("dtype,sum_mode", [("f32", "kahan32"), ("f64", "f64")])
@pytest.mark.parametrize("n_cat,rows,what", CASES)
def test_forms_and_groups(ara, n_cat, rows, what, dtype, sum_mode):
    from workloads import ELT, YET, Layer, Portfolio
    rng = np.random.default_rng(n_cat + len(rows) + rows[0])
    layers = []
    for u, n in enumerate(rows):
        n_rows = max(n, 1)
        ev = np.sort(rng.choice(n_cat, n_rows, replace=False)).astype(np.int32)
        m = np.exp(rng.normal(12, 1, n_rows)).astype(np.float32) + np.float32(2000.0)
        zero = np.zeros(n_rows, np.float32)
        elt = ELT(elt_id=u, event_ids=ev, mean=m, sigma_i=zero, sigma_c=zero, max_loss=2 * m,
                  retention=1e3, limit=1e9, share=0.9)
        # a layer of no paying event: the retention is above every loss
        layers.append(Layer(elts=[elt], occ_retention=0.0 if n else 1e12, occ_limit=1e9,
                            agg_retention=1e4 * (u + 1), agg_limit=1e12))
    pf = Portfolio(layers=layers, seed=5, su_enabled=False)
    lens = rng.integers(0, 1100, 8400)
    lens[:12] = [0, 1, 2, 3, 4, 5, 255, 256, 257, 1023, 1024, 1025]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    assert off[-1] >= 4_100_000
    yet = YET(offsets=off, event_ids=rng.integers(0, n_cat, off[-1]).astype(np.int32), times=None,
              n_catalogue=n_cat)
    print("forms", n_cat, rows, what, dtype, flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    kw = dict(ylt_dtype=dtype, sum_mode=sum_mode)
    r = ara.run(y, p, **kw)
    # a slice too small for the large tables
    s = ara.run(y, p, trial_count=3000, **kw)
    assert torch.equal(r["ylt"][:, :3000], s["ylt"]) and torch.equal(r["ylt_pf"][:3000], s["ylt_pf"])
    # the view's form of the passes (one layer each)
    v = ara.run(y, p, occ_view=True, **kw)
    assert torch.equal(r["ylt"], v["ylt"]) and torch.equal(r["ylt_pf"], v["ylt_pf"])
    # the layers one by one
    total = torch.zeros_like(r["ylt_pf"])
    for u in range(len(rows)):
        q = ara.load_portfolio(Portfolio(layers=[layers[u]], seed=5, su_enabled=False), n_cat)
        one = ara.run(y, q, **kw)["ylt"][0]
        assert torch.equal(one, r["ylt"][u])
        total = one if u == 0 else total + one
        ara.free_portfolio(q)
    assert torch.equal(total, r["ylt_pf"])
    n = 40
    few = YET(offsets=off[:n + 1], event_ids=yet.event_ids[:off[n]], times=None, n_catalogue=n_cat)
    ref = oracle.run_ara(few, pf, occ_view=True)
    G = ref["gross"]
    assert np.all(np.abs(r["ylt"][:, :n].double().cpu().numpy() - ref["ylt"]) <= 1e-5 * G + 1e-3)
    d = v["occ_view"][:, :off[n]].double().cpu().numpy()
    per_occ = np.repeat(G, np.diff(off[:n + 1]), axis=1)
    assert np.all(np.abs(d - ref["occ_view"]) <= 2 * (1e-5 * per_occ + 1e-3))
    ara.free_portfolio(p)
    ara.free_yet(y)
