"""PML/TVaR selection and the exceedance curve at the sizes where their form changes.

Losses are whole 64ths so that every sum is exact in FP64: PML, TVaR's sum and the
running means' sums are compared without a summation error, and what is left is one
rounding of a product, a sum and a quotient (4e-16, bounded by 1e-15).
"""
import numpy as np
import pytest

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


def losses(kind, n, dtype, rng):
    if kind == "wide":                       # every digit of the keys differs
        x = np.floor(np.exp(rng.uniform(-3, 15, n)) * 64) / 64
    elif kind == "ties":
        x = rng.choice([0.0, -0.0, 0.25, 3.0, 2.0 ** 18, 2.0 ** 18 + 0.25], n)
    else:
        x = np.full(n, 12345.25)
    return x.astype(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["wide", "ties", "equal"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4097, 16383, 16384, 16385, 32768, 32769,
                               65537, 300_007])
def test_select_and_sort(ara, n, kind, dtype):
    rng = np.random.default_rng(n)
    x = losses(kind, n, dtype, rng)
    ref = np.sort(np.abs(x).astype(np.float64))[::-1]
    print("select and sort", n, kind, dtype.__name__, flush=True)
    y = torch.from_numpy(x).cuda()
    srt, mean = ara.ep_curve(y)
    assert np.array_equal(srt.cpu().numpy().astype(np.float64), ref)
    assert not torch.signbit(srt).any()
    means = np.cumsum(ref) / np.arange(1, n + 1)
    assert np.all(np.abs(mean.cpu().numpy() - means) <= 1e-15 * means)
    assert torch.equal(ara.ep_curve(y, tail_mean=False)[0], srt)
    # one period, a full group, one more than a group, one more than two
    for m in (1, 16, 17, 33):
        rps = [1.0] + [float(r) for r in np.exp(rng.uniform(0, np.log(2.0 * n + 2), m - 1))]
        pml, tvar = ara.pml_tvar(y, rps)
        k = np.array([max(1, min(n, int(np.floor(n / rp)))) for rp in rps])
        got = np.asarray(pml.cpu() if hasattr(pml, "cpu") else pml, np.float64)
        tv = np.asarray(tvar.cpu() if hasattr(tvar, "cpu") else tvar, np.float64)
        assert np.array_equal(got, ref[k - 1])
        assert np.all(np.abs(tv - means[k - 1]) <= 1e-15 * means[k - 1])
