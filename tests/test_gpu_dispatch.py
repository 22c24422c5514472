"""The rules that choose between the point kernel, the far kernel and tiles over the whole window:
both sides of each line against the FP64 oracle (FP32 path: below 2e-6; FP64 path: its core, 8.5e-9,
below 2e-8), and the side taken, told from the bits: those of the tile kernel are the ones of
an explicit tile_group of 1."""
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


def _check(ctx, L, grid, pts, o, idx=None, tol=2e-6, rule="fixed"):
    """The call's rows, checked at grid[idx]."""
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    sig = ctx.compute(h, g, pts, o)
    idx = np.arange(len(grid)) if idx is None else idx
    for k, (P, T) in enumerate(pts):
        ref = O.sigma(L, grid, P, T, 16.0, cut_kind=rule, cut_cm1=o.cut_cm1, fwhm_mult=100.0,
                      points=idx)
        st = O.compare(sig[k][idx], ref, rel_tol=tol)
        assert st["violations"] == 0, (pts[k], st)
    ctx.unload_lines(h)
    ctx.free_grid(g)
    return sig


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,m,rows,moments", [
    (100_000, 200_000, 1, True), (100_000, 200_001, 1, False),   # 526 lines in a window
    (950_000, 200_001, 1, True),                                 # 5000 lines
    (950_000, 100_000, 10, True), (950_000, 100_000, 11, False),
])
def test_few_lines_many_points(ctx, n, m, rows, moments, f64):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(n, 500.0, 10000.0, 3))
    grid = 2000.0 + 0.005 * np.arange(m, dtype=np.float64)
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    idx = np.linspace(0, m - 1, 300).astype(np.int64)
    pts = [(0.1, 900.0 + k) for k in range(rows)]
    sig = _check(ctx, L, grid, pts, ctx.opts(0, 25.0, 100.0, prec), idx, 2e-8 if f64 else 2e-6)
    # by the tile kernel (a cut this wide groups tiles on the FP32 path) with any split
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    line = any(np.array_equal(sig, ctx.compute(h, g, pts, ctx.opts(
        0, 25.0, 100.0, prec, 2, split, tile_group=1 if f64 else 4))) for split in range(1, 65))
    assert line == (not moments and not f64)   # (FP64: at any size)
    ctx.unload_lines(h)
    ctx.free_grid(g)


def _chunk_list(kind):
    """Lists with more than two thousand lines in a window (FP64 tile kernel by chunks)."""
    if kind == "sparse":        # a chunk of 64 lines is 64 cm^-1 wide
        return synth.make_lines(synth.ListSpec(9000, 100.0, 9100.0, 17)), 2500.0
    L = synth.make_lines(synth.ListSpec(4200, 960.0, 1050.0, 17))
    rng = np.random.default_rng(17)
    if kind == "cluster":       # nearly all lines in one narrow band, a few thin ones around
        L["nu0"] = np.where(np.arange(4200) < 4160, 1011.0 + 0.02 * rng.random(4200), L["nu0"])
    elif kind == "short_cut":   # the cut splits chunks, rows and the tile
        L["nu0"] = 1000.0 + 2.0 * rng.random(4200)
    order = np.argsort(L["nu0"], kind="stable")
    return {k: v[order] for k, v in L.items()}, {"cluster": 25.0, "short_cut": 0.9}[kind]


@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
@pytest.mark.parametrize("kind", ["sparse", "cluster", "short_cut"])
def test_fp64_chunks(ctx, kind, rule):
    from paper_2510_20870_amd import xsec as X
    L, cut = _chunk_list(kind)
    grid = (3000.0 if kind == "sparse" else 1000.0) + 0.01 * np.arange(261, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(1e-4, 500.0), (0.3, 1500.0), (80.0, 700.0)]
    cutk = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    for P in (1, 2, 4):
        for split in (1, 3):
            o = ctx.opts(cutk, cut, 100.0, X.XS_FP64, P, split)
            full = ctx.compute(h, g, pts, o)
            o.select_eps = 1e-4
            part = ctx.compute(h, g, pts, o)
            for k, (p, t) in enumerate(pts):
                ref = O.sigma(L, grid, p, t, 16.0, cut_kind=rule, cut_cm1=cut, fwhm_mult=100.0)
                st = O.compare(full[k], ref, rel_tol=2e-8)
                assert st["violations"] == 0, (P, split, pts[k], st)
                assert np.all(part[k] <= ref * (1.0 + 2e-8)), (P, split, pts[k])
                assert np.all(part[k] >= ref * (1.0 - 1e-4 - 2e-8)), (P, split, pts[k])
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("m", [5, 13, 700])
def test_given_splits(ctx, m, f64):
    """A given split counts the parts of a tile of 64 points per lane; the point kernel's groups of
    8 points are parts of it already."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(40_000, 970.0, 1035.0, 91))
    grid = 1000.0 + 0.01 * np.arange(m, dtype=np.float64)
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    pts = [(0.3, 1500.0), (80.0, 700.0)]   # 0.3 bar: by the point kernel
    ref = [O.sigma(L, grid, p, t, 16.0, cut_cm1=25.0) for p, t in pts]
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    rows = {}
    for P in (1, 2):
        for split in (1, 2, 8, 9, 17, 256):
            sig = ctx.compute(h, g, pts, ctx.opts(0, 25.0, 100.0, prec, P, split))
            for k in range(2):
                st = O.compare(sig[k], ref[k], rel_tol=2e-8 if f64 else 2e-6)
                assert st["violations"] == 0, (P, split, pts[k], st)
            rows[P, split] = sig[0]
    ctx.unload_lines(h)
    ctx.free_grid(g)
    for P, split in ((1, 2), (1, 8), (1, 9), (2, 17)):
        c = min(8 * P, (m + 7) // 8)
        one = -(-split // c) == 1
        assert np.array_equal(rows[P, split], rows[P, 1]) == one, (P, split)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("kind", ["uniform", "gap"])
def test_broad_points_whatever_the_tile(ctx, kind, f64):
    """(P, T) points with broad lines go by tiles for every number of points per lane (ragged
    tiles, two points of which one is narrow), a gap at the grid's middle or not: rows against
    the oracle, and the same with more parts."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(60_000, 970.0, 1060.0, 91))
    grid = 1000.0 + 0.01 * np.arange(700, dtype=np.float64)
    if kind == "gap":
        grid[350:] += 20.0
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    pts = [(80.0, 700.0), (0.3, 1500.0), (100.0, 400.0)]
    ref = [O.sigma(L, grid, p, t, 16.0, cut_cm1=25.0) for p, t in pts]
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    for P in (1, 2, 4, 8):
        for split in (0, 1, 3):
            sig = ctx.compute(h, g, pts, ctx.opts(0, 25.0, 100.0, prec, P, split))
            for k in range(len(pts)):
                st = O.compare(sig[k], ref[k], rel_tol=2e-8 if f64 else 2e-6)
                print(f"[broad points] {kind} f64={f64} P={P} split {split} {pts[k]} "
                      f"max_rel {st['max_rel']:.2e}", flush=True)
                assert st["violations"] == 0, (P, split, pts[k], st)
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
def test_one_point(ctx, rule, f64):
    """Grids of one point, narrow and broad lines."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(60_000, 970.0, 1035.0, 91))
    kind = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    for nu in (1003.3, 946.0, 1020.25):
        for split in (0, 1, 5):
            o = ctx.opts(kind, 25.0, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=split)
            _check(ctx, L, np.array([nu]), [(1e-3, 500.0), (0.1, 900.0), (20.0, 800.0),
                                            (100.0, 400.0)], o, tol=2e-8 if f64 else 2e-6,
                   rule=rule)


def test_tuned_shapes_are_for_whole_windows(ctx):
    """A tuned shape changes the calls that walk whole windows; those by moments, also their broad
    points, keep their own."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(40_000, 970.0, 1035.0, 91))
    grid = 1000.0 + 0.01 * np.arange(900, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(0.3, 1500.0), (80.0, 700.0)]
    moments, walk = ctx.opts(0, 25.0), ctx.opts(0, 25.0, tile_group=1)
    try:
        a, b = ctx.compute(h, g, pts, moments), ctx.compute(h, g, pts, walk)
        X.tune_cache_put(ctx.tune_key(h, g, len(pts), moments), 4, 3, 16, 1.0)
        assert np.array_equal(ctx.compute(h, g, pts, moments), a)
        assert not np.array_equal(ctx.compute(h, g, pts, walk), b)
    finally:
        X.tune_cache_clear()
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("kind", ["uniform", "clusters", "coincident", "end", "past", "partners"])
def test_fwhm_by_moments(ctx, kind, f64):
    """FWHM cuts by moments (grids of 16384 points and more), as lists whose leaves and blocks are
    wide or narrow, lines with one centre, a last block that lacks a few lines, a grid past both
    ends, partners: at a sample of points, narrow to broad lines."""
    from paper_2510_20870_amd import xsec as X
    n, lo, hi, g0, step = {"end": (64 * 1024 - 5, 1000.0, 1012.0, 1001.0, 6e-4),
                           "past": (40_000, 1000.0, 1020.0, 985.0, 3e-3)}.get(
        kind, (60_000, 970.0, 1035.0, 1000.0, 3e-4))
    L = synth.make_lines(synth.ListSpec(n, lo, hi, 91))
    rng = np.random.default_rng(91)
    if kind == "clusters":
        c = lo + (hi - lo) * np.array([0.1, 0.42, 0.55, 0.9])
        L["nu0"] = np.where(rng.random(n) < 0.67, c[rng.integers(0, 4, n)] + 0.02 * rng.random(n),
                            L["nu0"])
    elif kind == "coincident":
        L["nu0"] = np.round(L["nu0"], 1)
    order = np.argsort(L["nu0"], kind="stable")
    L = {k: v[order] for k, v in L.items()}
    B = None
    if kind == "partners":
        L["J_low"], B = synth.j_low(L["E_low"]), synth.broadening_partners()
    m = 16_500
    grid = g0 + step * np.arange(m, dtype=np.float64)
    idx = np.unique(np.concatenate([rng.integers(0, m, 150), [0, m - 1], np.arange(800, 816)]))
    pts = [(1e-4, 500.0), (0.3, 1500.0), (3.0, 900.0), (80.0, 700.0)]
    h = ctx.load_lines(L, 16.0, broadening=B) if B else ctx.load_lines(L, 16.0)
    g = ctx.set_grid(grid)
    ref = [O.sigma(L, grid, p, t, 16.0, cut_kind="min_fwhm", cut_cm1=25.0, fwhm_mult=100.0,
                   points=idx, broadening=B) for p, t in pts]
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    for split in (0, 1, 17):
        sig = ctx.compute(h, g, pts, ctx.opts(X.XS_CUT_MIN_FWHM, 25.0, 100.0, prec, split=split))
        for k, r in enumerate(ref):
            st = O.compare(sig[k][idx], r, rel_tol=2e-8 if f64 else 2e-6)
            print(f"[fwhm] {kind} f64={f64} split {split} {pts[k]} max_rel {st['max_rel']:.2e}",
                  flush=True)
            assert st["violations"] == 0, (split, pts[k], st)
    walk = ctx.compute(h, g, pts, ctx.opts(X.XS_CUT_MIN_FWHM, 25.0, 100.0, prec, 2, 1,
                                           tile_group=1))
    assert not np.array_equal(walk[0], sig[0])
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
def test_grid_beyond_its_list(ctx, f64):
    """A grid whose middle lies far outside its list: the rule looks at the lines in reach."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(60_000, 1000.0, 1060.0, 4))
    grid = 1030.0 + 0.5 * np.arange(3000, dtype=np.float64)
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    o = ctx.opts(0, 25.0, 100.0, prec, 2, 1)
    sig = _check(ctx, L, grid, [(0.1, 900.0)], o, tol=2e-8 if f64 else 2e-6)
    o.tile_group = 1
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    assert not np.array_equal(ctx.compute(h, g, [(0.1, 900.0)], o), sig)
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("split", [0, 2])
def test_fp64_chunks_of_a_table(ctx, split):
    """FWHM cuts on the FP64 path: points whose lines' own cuts hold few lines and points with many,
    alone, in two runs and in turn; with a given split a row is that of its point alone."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(12_000, 990.0, 1030.0, 17))
    grid = 1008.0 + 0.004 * np.arange(333, dtype=np.float64)
    narrow, broad = (1e-3, 500.0), (8.0, 700.0)
    o = ctx.opts(X.XS_CUT_MIN_FWHM, 15.0, 100.0, X.XS_FP64, 2, split)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    ref = {p: O.sigma(L, grid, *p, 16.0, cut_kind="min_fwhm", cut_cm1=15.0, fwhm_mult=100.0)
           for p in (narrow, broad)}
    alone = {p: ctx.compute(h, g, [p], o)[0] for p in ref}
    for pts in ([narrow, broad], [broad] * 3 + [narrow] * 2, [narrow, broad] * 5):
        sig = ctx.compute(h, g, pts, o)
        for k, p in enumerate(pts):
            st = O.compare(sig[k], ref[p], rel_tol=2e-8)
            assert st["violations"] == 0, (k, p, st)
            if split:
                assert np.array_equal(sig[k], alone[p]), (k, p)
    # with selection: each run of points by its own thresholds
    o.split, o.select_eps = 2, 1e-3
    sel = ctx.compute(h, g, [broad, narrow, narrow, broad], o)
    for k, p in enumerate([broad, narrow, narrow, broad]):
        assert np.array_equal(sel[k], ctx.compute(h, g, [p], o)[0]), (k, p)
        assert np.all(sel[k] <= ref[p] * (1.0 + 2e-8)), (k, p)
        assert np.all(sel[k] >= ref[p] * (1.0 - 1e-3 - 2e-8)), (k, p)
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("n,m,P,f64,split,moments", [
    (27_000, 1349, 0.1, False, 0, False), (27_000, 1349, 8.0, False, 0, True),
    (27_000, 17_000, 1.0, False, 0, False), (60_000, 17_000, 0.1, False, 0, True),
    (60_000, 140_000, 0.1, False, 0, False), (60_000, 140_000, 8.0, False, 0, True),
    (120_000, 140_000, 0.1, False, 0, True),
    (27_000, 1349, 1.0, True, 0, False), (27_000, 1349, 8.0, True, 0, True),
    (27_000, 17_000, 0.1, True, 0, False), (60_000, 17_000, 0.1, True, 0, True),
    (27_000, 1349, 8.0, False, 3, False), (60_000, 1349, 0.1, False, 3, True)])
def test_fwhm_rule(ctx, n, m, P, f64, split, moments):
    """Both sides of the rule for FWHM cuts; the route shows in the bits (split 1: the automatic
    split of either is another one)."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(n, 970.0, 1030.0, 8))
    grid = 999.0 + (2.0 / m) * np.arange(m, dtype=np.float64)
    idx = np.unique(np.random.default_rng(8).integers(0, m, 60))
    o = ctx.opts(X.XS_CUT_MIN_FWHM, 25.0, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=split)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    sig = ctx.compute(h, g, [(P, 900.0)], o)[0]
    ref = O.sigma(L, grid, P, 900.0, 16.0, cut_kind="min_fwhm", cut_cm1=25.0, fwhm_mult=100.0,
                  points=idx)
    st = O.compare(sig[idx], ref, rel_tol=2e-8 if f64 else 2e-6)
    assert st["violations"] == 0, st
    o.tile_group = 1
    assert np.array_equal(ctx.compute(h, g, [(P, 900.0)], o)[0], sig) != moments
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
@pytest.mark.parametrize("split", [0, 2])
def test_points_that_go_different_ways(ctx, rule, split, f64):
    """Narrow and broad points alone, in runs and in turn (a small table goes one way as a whole),
    up to near ranges of the whole list; with a given split a row is that of its point alone."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(60_000, 1000.0, 1012.0, 23))
    # (three groups of points: two bands)
    kinds = [(0.01, 600.0), (4.0, 900.0), (30.0, 700.0), (100.0, 400.0)]
    for grid in (1003.0 + 0.002 * np.arange(400), np.concatenate(
            [1001.0 + 0.002 * np.arange(13), 1010.0 + 0.002 * np.arange(8)]), np.array([1006.0])):
        o = ctx.opts(X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM, 40.0, 100.0,
                     X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=split)
        h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
        ref = {p: O.sigma(L, grid, *p, 16.0, cut_kind=rule, cut_cm1=40.0, fwhm_mult=100.0)
               for p in kinds}
        alone = {p: ctx.compute(h, g, [p], o)[0] for p in kinds}
        for pts in (kinds, kinds[::-1], kinds * 3, [kinds[0], kinds[3]] * 5):
            sig = ctx.compute(h, g, pts, o)
            for k, p in enumerate(pts):
                st = O.compare(sig[k], ref[p], rel_tol=2e-8 if f64 else 2e-6)
                assert st["violations"] == 0, (len(grid), k, p, st)
                if split:
                    assert np.array_equal(sig[k], alone[p]), (len(grid), k, p)
        ctx.unload_lines(h)
        ctx.free_grid(g)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,m", [(900, 34_000), (900, 3000), (12_000, 34_000)])
def test_selection_workgroups(ctx, n, m, f64):
    """Thresholds by 4 waves (few lines, more than 64 groups of tiles), by 16: dropped lines stay
    within select_eps, and a row does not depend on the table with a given split."""
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(n, 1000.0, 1120.0, 6))
    grid = 1001.0 + 0.003 * np.arange(m, dtype=np.float64)
    idx = np.unique(np.random.default_rng(6).integers(0, m, 300))
    o = ctx.opts(X.XS_CUT_FIXED, 25.0, 100.0, X.XS_FP64 if f64 else X.XS_FP32_KAHAN, split=2,
                 select_eps=1e-3)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(0.05, 700.0), (20.0, 500.0)]
    sig = ctx.compute(h, g, pts, o)
    tol = 2e-8 if f64 else 2e-6
    for k, (P, T) in enumerate(pts):
        ref = O.sigma(L, grid, P, T, 16.0, points=idx)
        assert np.all(sig[k][idx] <= ref * (1.0 + tol)), (P, T)
        assert np.all(sig[k][idx] >= ref * (1.0 - 1e-3 - tol)), (P, T)
        assert np.array_equal(ctx.compute(h, g, [(P, T)], o)[0], sig[k])
    ctx.unload_lines(h)
    ctx.free_grid(g)
