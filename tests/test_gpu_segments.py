"""The quantile of shapes with a slot, at the edges of its polynomial segments.

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
