"""The point kernel at the edges of what its callers may pass, against the FP64 oracle: grid
points at and below zero, pressures so low that a profile's wing leaves FP32's range, gaps
between the points of a group.
Tolerances: the FP32 path's own error (K within 6e-7, sums below
1e-6, moments within 5e-8 of each contribution) stays below 2e-6; the FP64 path's core (8.5e-9)
below 2e-8."""
import numpy as np
import pytest

from oracle import xsec_oracle as O
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
@pytest.mark.parametrize("rule,lo,grid,pt,mult", [
    # the group from -4 to -2.25 holds a point at 2 v - 1 of its last one
    ("fixed", 0.01, -8.0 + 0.25 * np.arange(80), (0.1, 800.0), 100.0),
    ("min_fwhm", 0.01, -8.0 + 0.25 * np.arange(80), (1.0, 800.0), 100.0),
    # cuts of several times the line's own centre, so that lines close to zero reach no point
    # below it while those further up do
    ("min_fwhm", 0.001, -1.0 + 0.02 * np.arange(49), (1e-12, 1000.0), 1e6),
])
def test_points_below_zero(ctx, rule, lo, grid, pt, mult, f64):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(40_000, lo, 2.0 if lo < 0.01 else 20.0, 31))
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    ref = O.sigma(L, grid, pt[0], pt[1], 16.0, cut_kind=rule, cut_cm1=25.0, fwhm_mult=mult)
    kind = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    o = ctx.opts(kind, 25.0, mult, precision=X.XS_FP64 if f64 else X.XS_FP32_KAHAN)
    sig = ctx.compute(h, g, [pt], o)[0]
    assert np.all(np.isfinite(sig)), np.nonzero(~np.isfinite(sig))[0]
    st = O.compare(sig, ref, rel_tol=2e-8 if f64 else 2e-6)
    print(f"[below zero] {rule} f64={f64} max_rel {st['max_rel']:.2e}", flush=True)
    assert st["violations"] == 0, st
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("P", [1e-28, 1e-36, 1e-40])
def test_tiny_pressures(ctx, P):
    """Every point outside the Doppler cores (there the Lorentz wing is all there is, K down to
    1e-48), whatever its size beside the maximum."""
    n = 600
    L = synth.make_lines(synth.ListSpec(n, 1000.0, 1400.0, 5))
    grid = 1000.0 + 0.05 * np.arange(600, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    ref = O.sigma(L, grid, P, 800.0, 16.0, cut_cm1=25.0)
    sig = ctx.compute(h, g, [(P, 800.0)], ctx.opts(0, 25.0))[0]
    # 12 half-widths from every centre the Gaussian is below 1e-62
    b = O.doppler_width(grid, 800.0, 16.0)
    i = np.clip(np.searchsorted(L["nu0"], grid), 1, n - 1)
    wing = np.minimum(np.abs(grid - L["nu0"][i - 1]), np.abs(grid - L["nu0"][i])) > 12.0 * b
    rel = np.abs(sig - ref)[wing] / ref[wing]
    print(f"[tiny P] P={P} {int(wing.sum())} wing points max_rel {rel.max():.2e}", flush=True)
    assert rel.max() < 2e-6
    st = O.compare(sig, ref, rel_tol=2e-6)
    assert st["violations"] == 0, st
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
@pytest.mark.parametrize("split", [0, 1, 3])
def test_seams_of_a_grid(ctx, rule, split, f64):
    """Groups of points that span gaps of the grid: two bands that meet inside a group, a lone
    point between bands, gaps of just under and just over two cuts, steps wider than two cuts."""
    from paper_2510_20870_amd import xsec as X
    cut = 4.0
    L = synth.make_lines(synth.ListSpec(500_000, 1000.0, 1200.0, 12))
    grid = np.concatenate([1001.0 + 0.01 * np.arange(21), 1050.0 + 0.01 * np.arange(10), [1061.0],
                           1070.0 + 0.01 * np.arange(30), 1078.29 + 8.0 * np.arange(3),
                           1103.0 + 0.01 * np.arange(9) + 8.01 * np.arange(9), [1199.0, 1202.0]])
    pts = [(1e-3, 500.0), (0.3, 1500.0), (60.0, 700.0)]
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    kind = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    o = ctx.opts(kind, cut, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=split)
    sig = ctx.compute(h, g, pts, o)
    for k, (P, T) in enumerate(pts):
        ref = O.sigma(L, grid, P, T, 16.0, cut_kind=rule, cut_cm1=cut, fwhm_mult=100.0)
        st = O.compare(sig[k], ref, rel_tol=2e-8 if f64 else 2e-6)
        print(f"[seams] {rule} f64={f64} split {split} P={P} max_rel {st['max_rel']:.2e}",
              flush=True)
        assert st["violations"] == 0, (pts[k], st)
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("split", [0, 2])
def test_beyond_the_list(ctx, split, f64):
    """Points with no line in reach read 0, those at the edge of the cut do not; float32 and
    float64 rows."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(40_000, 1000.0, 1010.0, 12))
    grid = 985.0 + 0.03 * np.arange(2001, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    ref = O.sigma(L, grid, 0.1, 700.0, 16.0, cut_cm1=8.0)
    for out in (X.XS_F64, X.XS_F32):
        o = ctx.opts(0, 8.0, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=split,
                     out_dtype=out)
        sig = ctx.compute(h, g, [(0.1, 700.0)], o)[0].astype(np.float64)
        assert np.array_equal(sig == 0.0, ref == 0.0) and np.sum(ref == 0.0) > 500
        st = O.compare(sig, ref, rel_tol=2e-8 if f64 and out == X.XS_F64 else 2e-6)
        assert st["violations"] == 0, st
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n", [3000, 20_000, 400_000])
def test_gaps_of_few_lines(ctx, n, f64):
    """Two bands that meet inside a group and a step's widening, over gaps of less than 1024 lines,
    of more, and of more than 8192."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(n, 500.0, 1500.0, 12))
    grid = np.concatenate([600.0 + 0.01 * np.arange(1044), 900.0 + 0.01 * np.arange(90),
                           1000.0 + 30.0 * np.arange(17)])
    pts = [(0.01, 1500.0), (5.0, 600.0)]
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    sig = ctx.compute(h, g, pts, ctx.opts(X.XS_CUT_FIXED, 10.0, 0.0,
                                          X.XS_FP64 if f64 else X.XS_FP32_KAHAN))
    for k, (P, T) in enumerate(pts):
        ref = O.sigma(L, grid, P, T, 16.0, cut_cm1=10.0)
        st = O.compare(sig[k], ref, rel_tol=2e-8 if f64 else 2e-6)
        print(f"[gaps] n={n} f64={f64} P={P} max_rel {st['max_rel']:.2e}", flush=True)
        assert st["violations"] == 0, (pts[k], st)
    ctx.unload_lines(h)
    ctx.free_grid(g)
