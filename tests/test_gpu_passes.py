"""The passes of a run with secondary uncertainty give the same trial the same bits.

The pass is chosen by the size of the run and by its rows (``debug_run_pass``), so a
run, its slices, its diagnostic pass and a batch may each take another one."""
import pytest

from test_gpu_segments import table_case

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
