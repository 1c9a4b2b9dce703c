"""Portfolios loaded on streams other than the default one."""
import pytest

from workloads import Layer, Portfolio, make_elt, make_yet

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


def test_per_thread_stream(ara):
    """hipStreamPerThread means the calling thread's stream: a portfolio of more rows than
    all staging buffers together hold (4 MB), loaded on it behind work that keeps it
    busy, equals the one loaded on an ordinary stream."""
    from paper_1501_06326_amd.ara import (DevicePortfolio, _Desc, ara_load_portfolio,
                                          ara_portfolio_workspace_size, ara_run, ara_run_opts,
                                          ara_run_scratch_size, ara_sync_status)
    per_thread = 2                                   # hipStreamPerThread
    n_cat, n = 60_000, 500
    yet = make_yet(n, 300.0, n_cat, 7, with_times=False)
    pf = Portfolio(layers=[Layer(elts=[make_elt(e, 40_000, n_cat, e, retention=1e5, limit=5e7)
                                       for e in range(8)],
                                 occ_retention=1e5, occ_limit=2e8, agg_retention=1e6, agg_limit=1e12)],
                   seed=4)
    print("per-thread stream", flush=True)
    y = ara.load_yet(yet)
    p = ara.load_portfolio(pf, n_cat)
    ref = ara.run(y, p)["ylt_pf"]
    d = _Desc(pf)
    size = ara_portfolio_workspace_size(d.desc, n_cat)
    ws = torch.full((size,), 0, dtype=torch.uint8, device="cuda")
    scratch = torch.empty(ara_run_scratch_size(n), dtype=torch.uint8, device="cuda")
    out = torch.zeros(n, device="cuda")
    torch.cuda.synchronize()
    for _ in range(3):
        # earlier runs on the stream are still going when the load's copies are enqueued
        o = ara_run_opts(trial_count=n, d_scratch=scratch.data_ptr(), scratch_bytes=scratch.numel())
        for _ in range(20):
            ara_run(ara.ctx, y.handle, p.handle, o, None, out.data_ptr(), per_thread)
        h = ara_load_portfolio(ara.ctx, d.desc, n_cat, ws.data_ptr(), size, per_thread)
        q = DevicePortfolio(h, ws, 1, pf.n_elts, True)
        out.zero_()
        torch.cuda.synchronize()
        ara_run(ara.ctx, y.handle, q.handle, o, None, out.data_ptr(), per_thread)
        ara_sync_status(ara.ctx, per_thread)
        assert torch.equal(out, ref)
        ara.free_portfolio(q)
    ara.free_portfolio(p)
    ara.free_yet(y)


@pytest.mark.parametrize("rows", [1, 32_767, 32_768, 32_769, 52_428, 52_429, 120_000])
def test_rows_by_size(ara, rows):
    """Rows copied from the caller's array (up to 32,768), from one buffer and from
    several: split over two ELTs of one layer, every row arrives (the diagnostic pass
    counts a hit for each, once per event of a YET that visits every event)."""
    import numpy as np
    from workloads import ELT, YET
    n_cat = 70_000
    elts, left = [], rows
    for e in range(2):
        n = (rows + 1) // 2 if e == 0 else left
        left -= n
        ev = np.arange(n, dtype=np.int32)
        m = np.full(n, 1e5, np.float32) + np.arange(n, dtype=np.float32)
        zero = np.zeros(n, np.float32)
        elts.append(ELT(elt_id=e, event_ids=ev, mean=m, sigma_i=zero, sigma_c=zero, max_loss=2 * m,
                        retention=0.0, limit=1e12, share=1.0))
    inf = float("inf")
    pf = Portfolio(layers=[Layer(elts=elts, occ_retention=0.0, occ_limit=inf, agg_retention=0.0,
                                 agg_limit=inf)], seed=1)
    off = np.arange(0, n_cat + 1, 70, dtype=np.int64)
    yet = YET(offsets=off, event_ids=np.arange(n_cat, dtype=np.int32), times=None, n_catalogue=n_cat)
    print("rows by size", rows, flush=True)
    y = ara.load_yet(yet)
    for _ in range(2):
        p = ara.load_portfolio(pf, n_cat)
        d = ara.run(y, p, diagnostics=True, sum_mode="f64", ylt_dtype="f64")
        per_event = np.zeros(n_cat)
        hits = np.zeros(n_cat, np.int64)
        for e in elts:
            np.add.at(per_event, e.event_ids, e.mean.astype(np.float64))
            np.add.at(hits, e.event_ids, 1)
        assert np.array_equal(d["hits"][0].cpu().numpy(), hits.reshape(-1, 70).sum(axis=1))
        # two FP32 losses an event are added in FP32
        want = per_event.reshape(-1, 70).sum(axis=1)
        assert np.all(np.abs(d["ylt"][0].cpu().numpy() - want) <= 2.0 ** -24 * want)
        ara.free_portfolio(p)
    ara.free_yet(y)
