"""The far field by moments of line groups (far.hip) against the FP64 oracle where it can go
wrong: ragged tiles and leaves, a grid that reaches past the list, cuts that end inside a
leaf or inside the tile, lists whose leaves are wide (sparse) beside narrow ones (clusters),
coincident centres, lines so broad that no group is far, and too little memory for the
moments. Tolerances: the FP32 path's own error (K within 6e-7, sums below 1e-6, moments
within 5e-8 of each contribution) stays below 2e-6; the FP64 path's core (8.5e-9) below 2e-8."""
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


def _lists(kind, n, lo, hi, seed):
    L = synth.make_lines(synth.ListSpec(n, lo, hi, seed))
    rng = np.random.default_rng(seed)
    if kind == "clusters":
        # two thirds of the lines in four narrow bands, the rest spread thinly
        m = rng.random(n) < 0.67
        c = lo + (hi - lo) * np.array([0.1, 0.42, 0.55, 0.9])
        L["nu0"] = np.where(m, c[rng.integers(0, 4, n)] + 0.02 * rng.random(n), L["nu0"])
    elif kind == "coincident":
        L["nu0"] = np.round(L["nu0"], 1)
    order = np.argsort(L["nu0"], kind="stable")
    return {k: v[order] for k, v in L.items()}


# name: list kind, lines, list range, grid (start, step, points), cut
CASES = {
    "ragged": ("uniform", 60_000, (970.0, 1035.0), (1000.0, 0.01, 5 * 64 + 1), 25.0),
    "past_ends": ("uniform", 40_000, (1000.0, 1020.0), (985.0, 0.25, 200), 25.0),
    "one_point": ("uniform", 60_000, (970.0, 1035.0), (1003.3, 0.01, 1), 25.0),
    "clusters": ("clusters", 50_000, (970.0, 1035.0), (997.0, 0.02, 390), 25.0),
    "coincident": ("coincident", 50_000, (970.0, 1035.0), (1000.0, 0.015, 260), 25.0),
    "short_cut": ("uniform", 90_000, (1000.0, 1004.0), (1001.0, 0.02, 100), 0.6),
    "wide_tiles": ("uniform", 60_000, (970.0, 1035.0), (980.0, 0.4, 130), 25.0),
    # the FWHM cut: from a few Doppler widths over cuts that differ by line to the common cap
    "fwhm": ("uniform", 60_000, (970.0, 1035.0), (1000.0, 0.01, 5 * 64 + 1), 25.0),
    "fwhm_clusters": ("clusters", 50_000, (970.0, 1035.0), (997.0, 0.02, 390), 25.0),
    # dense lists, whole blocks of 1024 lines between the smallest and the largest cut; the
    # last block of the second lacks a few lines
    "fwhm_blocks": ("uniform", 120_000, (990.0, 1030.0), (1005.0, 0.003, 150), 25.0),
    "fwhm_block_end": ("uniform", 64 * 1024 - 5, (1000.0, 1012.0), (1001.0, 0.05, 200), 25.0),
    "fwhm_past_ends": ("coincident", 40_000, (1000.0, 1020.0), (985.0, 0.25, 200), 25.0),
}


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("case", sorted(CASES))
def test_moments_vs_oracle(ctx, case, f64):
    from paper_2510_20870_amd import xsec as X
    kind, n, (lo, hi), (g0, step, m), cut = CASES[case]
    L = _lists(kind, n, lo, hi, 91)
    grid = g0 + step * np.arange(m, dtype=np.float64)
    h = ctx.load_lines(L, 16.0)
    g = ctx.set_grid(grid)
    pts = [(1e-4, 500.0), (0.3, 1500.0), (80.0, 700.0)]
    fwhm = case.startswith("fwhm")
    if fwhm:
        pts.append((3.0, 900.0))
    rule = "min_fwhm" if fwhm else "fixed"
    ref = [O.sigma(L, grid, P, T, 16.0, cut_kind=rule, cut_cm1=cut, fwhm_mult=100.0)
           for P, T in pts]
    kind = X.XS_CUT_MIN_FWHM if fwhm else X.XS_CUT_FIXED
    prec = X.XS_FP64 if f64 else X.XS_FP32_KAHAN
    for split in (0, 1, 3):
        o = ctx.opts(kind, cut, 100.0, precision=prec, split=split)
        sig = ctx.compute(h, g, pts, o)
        for k, r in enumerate(ref):
            st = O.compare(sig[k], r, rel_tol=2e-8 if f64 else 2e-6)
            print(f"[moments] {case} f64={f64} P={pts[k][0]} split {split} "
                  f"max_rel {st['max_rel']:.2e}", flush=True)
            assert st["violations"] == 0, st
        assert np.array_equal(ctx.compute(h, g, pts, o), sig)   # bitwise repeatable
    # one point of the batch alone gives the same bits
    o = ctx.opts(kind, cut, 100.0, precision=prec, split=1)
    assert np.array_equal(ctx.compute(h, g, pts[1:2], o)[0], ctx.compute(h, g, pts, o)[1])
    ctx.unload_lines(h)
    ctx.free_grid(g)


def test_moments_fwhm_partners(ctx):
    """Broadening partners: the bounds of the cut come from the partners' tables."""
    from paper_2510_20870_amd import xsec as X
    L = _lists("uniform", 60_000, 970.0, 1035.0, 93)
    L["J_low"] = synth.j_low(L["E_low"])
    B = synth.broadening_partners()
    grid = 1000.0 + 0.015 * np.arange(200, dtype=np.float64)
    pts = [(1e-3, 800.0), (0.5, 1500.0), (20.0, 600.0)]
    h = ctx.load_lines(L, 16.0, broadening=B)
    g = ctx.set_grid(grid)
    sig = ctx.compute(h, g, pts, ctx.opts(X.XS_CUT_MIN_FWHM, 25.0, 100.0))
    for k, (P, T) in enumerate(pts):
        ref = O.sigma(L, grid, P, T, 16.0, cut_kind="min_fwhm", cut_cm1=25.0, fwhm_mult=100.0,
                      broadening=B)
        st = O.compare(sig[k], ref, rel_tol=2e-6)
        print(f"[moments] partners P={P} max_rel {st['max_rel']:.2e}", flush=True)
        assert st["violations"] == 0, st
    ctx.unload_lines(h)
    ctx.free_grid(g)


def test_moments_entry_points_agree(ctx):
    """Graph replay, the allocation-free call and a served request with the same explicit
    shape give xs_compute's bits; a budget that holds the records but not the moments still
    computes (line by line)."""
    import torch
    from paper_2510_20870_amd import xsec as X
    L = _lists("uniform", 60_000, 970.0, 1035.0, 92)
    grid = 1000.0 + 0.01 * np.arange(700, dtype=np.float64)
    pts = [(0.01, 900.0), (5.0, 1500.0)]
    h = ctx.load_lines(L, 16.0)
    g = ctx.set_grid(grid)
    o = ctx.opts(X.XS_CUT_FIXED, 25.0, split=2)
    want = ctx.compute(h, g, pts, o)
    out = torch.empty((2, 700), dtype=torch.float64, device="cuda")
    gr = ctx.graph_create(h, g, pts, o, out)
    for _ in range(3):
        out.fill_(-1.0)
        gr.launch(torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
        ctx.compute(h, g, pts[:1], o)
    gr.close()
    out.fill_(-1.0)
    ctx.compute_noalloc(h, g, pts, o, out, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    ctx.serve_start(mem_bytes=64 << 20)
    r = ctx.submit(h, g, pts, o)
    assert np.array_equal(r.wait(60.0), want)
    r.release()
    # list 1.56 MB + grid; one point's records are 1.7 MB, its moments 0.7 MB more
    small = X.Context(0, hbm_budget_bytes=3_560_000)
    hs = small.load_lines(L, 16.0)
    gs = small.set_grid(grid)
    o1 = ctx.opts(X.XS_CUT_FIXED, 25.0, split=1, out_dtype=X.XS_F32)
    out32 = torch.empty((1, 700), dtype=torch.float32, device="cuda")
    small.compute(hs, gs, pts[:1], o1, out=out32, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    used, budget = small.memory_used()
    assert budget - used < 400_000   # the moments need 0.7 MB (13 bytes per line)
    st = O.compare(out32.cpu().numpy()[0].astype(np.float64), want[0], rel_tol=2e-6)
    assert st["violations"] == 0, st
    small.close()
    ctx.unload_lines(h)
    ctx.free_grid(g)
