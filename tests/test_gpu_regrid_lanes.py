"""Bin means by 1, 4, 16 and 64 lanes per bin and 1 to 9 rows against the oracle's: bins of no
node, one node and many, nodes on a bin's ends, bins outside the source range, uneven source
steps. Tolerance: sums of at most 7e3 positive terms and bin widths of at least 1e-3 at 1e3 in
FP64 stay below 1e-9."""
import numpy as np
import pytest

from oracle import xsec_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_20870_amd import xsec
    ctx = xsec.Context(0)
    yield xsec, ctx
    ctx.close()


@pytest.mark.parametrize("n_src,n_dst,rows", [(257, 900, 1), (300, 299, 5), (1000, 400, 4),
                                              (1999, 401, 9), (2000, 61, 3), (7001, 31, 4),
                                              (7000, 2, 5), (2, 7, 2), (700, 1, 6)])
@pytest.mark.parametrize("uneven", [False, True])
def test_bin_means_by_lanes(env, n_src, n_dst, rows, uneven):
    X, ctx = env
    rng = np.random.default_rng(n_src + n_dst)
    x = 1000.0 + 10.0 * np.arange(n_src) / (n_src - 1)
    if uneven:
        x = 1000.0 + 10.0 * ((x - 1000.0) / 10.0) ** 3 if n_src == 2 else np.unique(
            1000.0 + 10.0 * ((x - 1000.0) / 10.0) ** 1.5)
    d = np.linspace(998.5, 1011.0, n_dst) if n_dst > 1 else np.array([1004.0])
    if n_dst > 30:   # some bin ends on nodes
        d[10:14] = 0.5 * (x[n_src // 3] + x[n_src // 3 + 1]) + 1e-2 * np.arange(4)
        d = np.unique(d)
    y = rng.uniform(1.0, 2.0, (rows, len(x)))
    gs, gd = ctx.set_grid(x), ctx.set_grid(d)
    got = ctx.regrid(gs, gd, y, X.XS_REGRID_BIN_MEAN)
    lin = ctx.regrid(gs, gd, y, X.XS_REGRID_LINEAR)
    for r in range(rows):
        np.testing.assert_allclose(got[r], O.regrid_bin_mean(d, x, y[r]), rtol=1e-9, atol=0)
        np.testing.assert_allclose(lin[r], O.regrid_linear(d, x, y[r]), rtol=1e-9, atol=0)
    ctx.free_grid(gs)
    ctx.free_grid(gd)
