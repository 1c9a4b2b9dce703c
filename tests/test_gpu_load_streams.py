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
