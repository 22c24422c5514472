"""Served requests by moments. Work items of broad lines: at most 4096 lines each, as for the
others (the number of parts is told from the bits of calls with that split given). Order: the
request with the least work left goes first, a request by moments counting what it costs."""
import numpy as np
import pytest

from oracle import xsec_oracle as O
from paper_2510_20870_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_20870_amd import xsec
    c = xsec.Context(0)
    yield c
    c.close()


def test_broad_requests_in_short_items(ctx):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(130_000, 970.0, 1035.0, 5))
    grid = 1000.0 + 0.01 * np.arange(512, dtype=np.float64)
    # 2000 points of 8 tiles are more than two rounds of wavefronts, so nothing but the item's
    # length asks for parts
    pts = [(100.0, 300.0 + 0.01 * k) for k in range(2000)]
    h, g = ctx.load_lines(L, 16.0), ctx.set_grid(grid)
    ctx.serve_start(mem_bytes=8 << 30)
    r = ctx.submit(h, g, pts, ctx.opts(X.XS_CUT_FIXED, 25.0))
    sig = r.wait(60.0)
    r.release()
    gmax = float(np.max(O.lorentz_width(L["gamma"], L["n_T"], 100.0, 300.0)))
    mid = grid[len(grid) // 2]
    near = int(np.sum(np.abs(L["nu0"] - mid) <= min(25.0, 3.5 * gmax)))
    parts = [s for s in range(1, 65) if np.array_equal(
        ctx.compute(h, g, pts[:1], ctx.opts(X.XS_CUT_FIXED, 25.0, pts_per_lane=1, split=s))[0],
        sig[0])]
    print(f"[items] {near} near lines, parts {parts}", flush=True)
    assert parts and min(parts) * 4096 >= near
    ref = O.sigma(L, grid, pts[-1][0], pts[-1][1], 16.0, cut_cm1=25.0)
    st = O.compare(sig[-1], ref, rel_tol=2e-6)
    assert st["violations"] == 0, st
    ctx.unload_lines(h)
    ctx.free_grid(g)


def test_least_work_first(ctx):
    from paper_2510_20870_amd import xsec as X
    L = synth.make_lines(synth.ListSpec(600_000, 970.0, 1130.0, 5))
    h = ctx.load_lines(L, 16.0)
    ctx.serve_start(max_inflight=1, mem_bytes=4 << 30, paused=True)
    pts = [(0.1, 900.0)]
    # selection walks all 190000 lines of every window; the full sum on four times the points
    # goes by moments and takes a tenth of the time
    slow = ctx.submit_window(h, 1030.0, 0.002, 10_000, pts,
                             ctx.opts(X.XS_CUT_FIXED, 25.0, select_eps=1e-4))
    fast = ctx.submit_window(h, 1030.0, 0.0005, 40_000, pts, ctx.opts(X.XS_CUT_FIXED, 25.0))
    ctx.serve_pause(False)
    a, b = slow.wait(60.0), fast.wait(60.0)
    assert np.all(np.isfinite(a)) and np.all(np.isfinite(b))
    t_slow, t_fast = slow.times(), fast.times()
    print(f"[order] slow {t_slow} fast {t_fast}", flush=True)
    assert t_fast[2] < t_slow[2]
    slow.release()
    fast.release()
    ctx.unload_lines(h)
