"""With a given split, a row has the bits of its own single-point call, whatever other points
stand beside it: windows below and above the limit of the far field by moments, narrow and broad
lines mixed, both cuts and precisions."""
import numpy as np
import pytest

from paper_2510_20870_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_20870_amd import xsec
    c = xsec.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
@pytest.mark.parametrize("n", [6500, 40_000])   # 5000 and 30000 lines within the cut
def test_rows_alone(ctx, n, rule, f64):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(n, 970.0, 1035.0, 7))
    grid = 1000.0 + 0.01 * np.arange(500, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    # enough narrow points that the call as a whole is a large one
    pts = [(0.1, 900.0), (100.0, 800.0), (1e-3, 500.0)] + [(0.01, 600.0 + k) for k in range(300)]
    kind = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    for P, split in ((0, 1), (0, 3), (2, 2), (4, 1)):
        o = ctx.opts(kind, 25.0, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, P, split)
        sig = ctx.compute(h, g, pts, o)
        for k in (0, 1, 2, 150):
            one = ctx.compute(h, g, pts[k:k + 1], o)[0]
            assert np.array_equal(one, sig[k]), (P, split, pts[k],
                                                 float(np.max(np.abs(one / sig[k] - 1.0))))
    ctx.unload_lines(h)
    ctx.free_grid(g)
