"""FP32 tile kernel: lines so broad that they enter a tile's polynomial from beside the tile or
from inside it, next to narrower ones, on whole and ragged tiles, against the FP64 oracle.
Tolerances: each line within the error budget (2e-7, or 1e-5 where that is asked for) plus
FP32 sums below 1e-6."""
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


@pytest.mark.parametrize("tol", [0.0, 1e-5])
@pytest.mark.parametrize("step,m", [(0.002, 64), (0.01, 321), (0.05, 700)])
def test_broad_lines_vs_oracle(ctx, step, m, tol):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(3000, 985.0, 1025.0, 23))
    grid = 1000.0 + step * np.arange(m, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(0.5, 700.0), (5.0, 1500.0), (30.0, 600.0), (100.0, 300.0)]
    ref = [O.sigma(L, grid, P, T, 16.0, cut_kind="fixed", cut_cm1=25.0) for P, T in pts]
    for P in (1, 2, 4, 8):
        o = ctx.opts(X.XS_CUT_FIXED, 25.0, pts_per_lane=P, split=2, tol=tol)
        sig = ctx.compute(h, g, pts, o)
        for k, r in enumerate(ref):
            st = O.compare(sig[k], r, rel_tol=tol + 2e-6)
            print(f"[broad] step {step} P={P} p={pts[k][0]} max_rel {st['max_rel']:.2e}", flush=True)
            assert st["violations"] == 0, (P, pts[k], st)
    ctx.unload_lines(h)
    ctx.free_grid(g)
