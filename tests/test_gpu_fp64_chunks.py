"""The FP64 path's tile kernel where a chunk of 64 lines enters a row of the tile by its
moments: rows of which some are far and some not, rows that a cut splits, short and ragged
chunks, wide chunks (sparse lists), cuts that differ by line, lines too broad for any row to be
far, with and without main-contributor selection. Tolerances: the FP64 path's core (8.5e-9)
below 2e-8; selection drops at most eps of sigma (lines dropped only lower it)."""
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


# name: lines, list range, grid (start, step, points), cut
CASES = {
    "ordinary": (6000, (970.0, 1035.0), (1000.0, 0.01, 5 * 64 + 1), 25.0),
    "sparse": (300, (960.0, 1050.0), (1000.0, 0.01, 200), 25.0),
    "few": (15, (999.0, 1003.0), (1000.0, 0.01, 130), 25.0),
    "short_cut": (3000, (995.0, 1010.0), (1000.0, 0.02, 300), 1.5),
    "past_ends": (3000, (1000.0, 1010.0), (985.0, 0.25, 150), 25.0),
}


@pytest.mark.parametrize("rule", ["fixed", "min_fwhm"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_chunks_vs_oracle(ctx, case, rule):
    from paper_2510_20870_amd import xsec as X
    n, (lo, hi), (g0, step, m), cut = CASES[case]
    L = synth.make_lines(synth.ListSpec(n, lo, hi, 17))
    grid = g0 + step * np.arange(m, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(1e-4, 500.0), (0.3, 1500.0), (80.0, 700.0)]
    kind = X.XS_CUT_FIXED if rule == "fixed" else X.XS_CUT_MIN_FWHM
    ref = [O.sigma(L, grid, P, T, 16.0, cut_kind=rule, cut_cm1=cut, fwhm_mult=100.0)
           for P, T in pts]
    for P in (1, 2, 4):
        for split in (1, 3):
            full = ctx.compute(h, g, pts, ctx.opts(kind, cut, 100.0, precision=X.XS_FP64,
                                                   pts_per_lane=P, split=split))
            part = ctx.compute(h, g, pts, ctx.opts(kind, cut, 100.0, precision=X.XS_FP64,
                                                   pts_per_lane=P, split=split,
                                                   select_eps=1e-4))
            for k, r in enumerate(ref):
                st = O.compare(full[k], r, rel_tol=2e-8)
                assert st["violations"] == 0, (P, split, pts[k], st)
                assert np.all(part[k] <= r * (1.0 + 2e-8)), (P, split, pts[k])
                assert np.all(part[k] >= r * (1.0 - 1e-4 - 2e-8)), (P, split, pts[k])
    ctx.unload_lines(h)
    ctx.free_grid(g)
