"""The mean of the quantile of shapes with a slot.

A Year Loss Table's means (TVaR, the expected loss) average millions of draws, so an
error that all draws of a segment share stays in them.  65,536 stratified draws of a
shape against the FP64 oracle's inverse: a draw's own rounding, up to 2.4e-7 of
max(root, mean) either way, averages to 1e-9 at most by chance (2.4e-7 / sqrt(65,536));
coefficients rounded so that a segment's mean is kept leave 4e-10 (rounded one by one,
1e-8).  Bound: 2e-9 of the mean.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b", [(2.75, 8.25), (1.5, 6.0), (32.0, 32.0), (12.0, 3.0), (1.0, 32.0)])
def test_mean_of_draws(a, b):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1501_06326_amd import Ara
    n = 1 << 16
    j = (np.arange(n, dtype=np.int64) << 8) + 2 * np.random.default_rng(3).integers(0, 128, n) + 1
    z, zc = j / 2.0 ** 24, ((1 << 24) - j) / 2.0 ** 24
    ara = Ara(0)
    print("mean quantile", a, b, flush=True)
    x, path = ara.debug_beta_quantile_shape(a, b, z, zc)
    ara.close()
    assert np.all(path == 0)
    ref = oracle.betaincinv(a, b, z, zc)
    off = float(np.mean(x.astype(np.float64) - ref)) / (a / (a + b))
    print("off by", off, flush=True)
    assert abs(off) <= 2e-9
