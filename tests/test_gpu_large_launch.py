"""Calls whose kernels take more than 2^32 threads: many grid points times many (P, T) points in
one batch. The last row has the bits of its own call (explicit shape), and a sample of points
agrees with the FP64 oracle (FP32 path: below 2e-6)."""
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


# name: lines, list's end, grid step, (P, T) points (2^21 grid points each), pressure, selection.
# Threads per grid point: point kernel 8, far kernel 4 (lines broad beside 384 grid steps),
# thresholds of the selection 4 (1 point per lane)
CASES = {
    "point": (180_000, 1470.0, 2e-4, 257, 0.1, 0.0),
    "far": (42_000, 1071.0, 1e-5, 513, 100.0, 0.0),
    "select": (40, 1071.0, 1e-5, 513, 0.1, 1e-4),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_more_than_2_32_threads(ctx, case):
    import torch
    from paper_2510_20870_amd import xsec as X
    n, hi, step, rows, P, eps = CASES[case]
    m = 1 << 21
    L = synth.make_lines(synth.ListSpec(n, 950.0, hi, 3))
    grid = 1000.0 + step * np.arange(m, dtype=np.float64)
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    pts = [(P * (1.0 + 1e-3 * k), 900.0) for k in range(rows)]
    o = ctx.opts(X.XS_CUT_FIXED, 25.0, 100.0, X.XS_FP32_KAHAN, 1, 1, 0, eps, X.XS_F32)
    out = torch.full((rows, m), -1.0, dtype=torch.float32, device="cuda")
    ctx.compute(h, g, pts, o, out=out, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert bool((out.amin(dim=1) > 0.0).all())
    one = torch.full((1, m), -1.0, dtype=torch.float32, device="cuda")
    ctx.compute(h, g, pts[-1:], o, out=one, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert bool((one[0] == out[-1]).all())
    idx = np.linspace(0, m - 1, 40).astype(np.int64)
    for k in (0, rows // 2, rows - 1):
        ref = O.sigma(L, grid, pts[k][0], pts[k][1], 16.0, cut_cm1=25.0, points=idx)
        got = out[k].cpu().numpy()[idx].astype(np.float64)
        st = O.compare(got, ref, rel_tol=2e-6 + eps)
        print(f"[large launch] {case} row {k} max_rel {st['max_rel']:.2e}", flush=True)
        assert st["violations"] == 0, st
    del out
    ctx.unload_lines(h)
    ctx.free_grid(g)
