"""The tile kernel over whole windows (tile_group 1, FP32 path), whatever the automatic choice takes
for such lists: its power-of-two scale over the range of magnitudes, every launch shape, lines at
the switch between the tile polynomial and the per-point forms from low to high pressure, lines
that enter the polynomial by their width. Against the FP64 oracle; tolerance 2e-6 (each line
within 6e-7 or its far form's 7e-7, FP32 sums below 1e-6), and 1e-5 more where the error budget is
1e-5."""
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


def _rows(ctx, L, grid, pts, shapes, cut=25.0, tol=0.0, mass=16.0, label=""):
    h, g = ctx.load_lines(L, mass), ctx.set_grid(grid)
    ref = [O.sigma(L, grid, P, T, mass, cut_cm1=cut) for P, T in pts]
    for P, split, W in shapes:
        o = ctx.opts(0, cut, 100.0, 0, P, split, W, tile_group=1, tol=tol)
        sig = ctx.compute(h, g, pts, o)
        assert np.all(np.isfinite(sig))
        for k, r in enumerate(ref):
            st = O.compare(sig[k], r, rel_tol=tol + 2e-6)
            print(f"[tile window] {label} {P, split, W} {pts[k]} max_rel {st['max_rel']:.2e}",
                  flush=True)
            assert st["violations"] == 0, (P, split, W, pts[k], st)
        assert np.array_equal(ctx.compute(h, g, pts, o), sig)
    ctx.unload_lines(h)
    ctx.free_grid(g)


@pytest.mark.parametrize("factor", [1e30, 1e-30])
def test_magnitudes(ctx, factor):
    L = synth.make_lines(synth.ListSpec(5000, 1500.0, 1520.0, 4))
    L["A"] = (L["A"].astype(np.float64) * factor).astype(np.float32)
    # strong lines late in the window, so that running sums are rescaled
    L["A"][4000::50] *= np.float32(1e4)
    grid = synth.uniform_grid(1499.0, 1521.0, 0.01)
    _rows(ctx, L, grid, [(0.02, 800.0), (5.0, 400.0)], [(1, 1, 0), (2, 3, 0), (8, 1, 0)], cut=3.0,
          mass=20.0, label=f"x{factor:g}")


def test_launch_shapes(ctx):
    L = synth.make_lines(synth.ListSpec(4000, 995.0, 1015.0, 9))
    grid = 1000.0 + 0.01 * np.arange(700, dtype=np.float64)
    shapes = [(P, split, W) for P in (1, 2, 4, 8) for split, W in ((1, 0), (7, 0), (3, 2))]
    shapes += [(P, 2, W) for P in (1, 2) for W in (3, 4, 5, 6)]
    _rows(ctx, L, grid, [(1e-3, 500.0), (1.0, 1500.0)], shapes, cut=10.0, label="shapes")


@pytest.mark.parametrize("tol,kappa", [(0.0, 4.09), (1e-5, 3.16)])
@pytest.mark.parametrize("gridkind", ["uniform", "ln"])
def test_far_switch(ctx, gridkind, tol, kappa):
    if gridkind == "uniform":
        grid = 1000.0 + 0.01 * np.arange(3 * 128 + 1, dtype=np.float64)
    else:
        grid = np.exp(np.linspace(np.log(990.0), np.log(1010.0), 2 * 128 + 37))
    base = synth.make_lines(synth.ListSpec(20_000, grid[0] - 30.0, grid[-1] + 30.0, 62))
    rng = np.random.default_rng(61)
    for P, T in ((0.1, 1500.0), (10.0, 300.0), (100.0, 500.0)):
        # 64 lines around kappa h + 1.25 b_D on both sides of every 128-point tile
        kb, extra = O.doppler_width(1.0, T, 16.0), []
        for j0 in range(0, len(grid), 128):
            t = grid[j0:j0 + 128]
            nc, hw = 0.5 * (t[0] + t[-1]), 0.5 * (t[-1] - t[0])
            for c in ((nc - kappa * hw) / (1.0 + 1.25 * kb), (nc + kappa * hw) / (1.0 - 1.25 * kb)):
                extra.append(c * (1.0 + rng.uniform(-1e-9, 1e-9, 64)))
        extra = np.concatenate(extra)
        src = rng.integers(0, len(base["nu0"]), len(extra))
        L = {k: np.concatenate([v, extra if k == "nu0" else v[src]]) for k, v in base.items()}
        order = np.argsort(L["nu0"], kind="stable")
        L = {k: v[order] for k, v in L.items()}
        _rows(ctx, L, grid, [(P, T)], [(2, 1, 0), (1, 3, 0), (4, 1, 0)], tol=tol,
              label=f"switch {gridkind}")


@pytest.mark.parametrize("step,m", [(0.002, 64), (0.01, 321), (0.05, 700)])
def test_broad_lines(ctx, step, m):
    L = synth.make_lines(synth.ListSpec(3000, 985.0, 1025.0, 23))
    grid = 1000.0 + step * np.arange(m, dtype=np.float64)
    pts = [(0.5, 700.0), (5.0, 1500.0), (30.0, 600.0), (100.0, 300.0)]
    for tol in (0.0, 1e-5):
        _rows(ctx, L, grid, pts, [(P, 2, 0) for P in (1, 2, 4, 8)], tol=tol, label=f"broad {step}")
