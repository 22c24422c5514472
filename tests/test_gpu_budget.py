"""Calls under a tight HBM budget: what fits line by line is computed, whatever the moments of
the far field would need and whatever earlier calls have left."""
import numpy as np
import pytest

from oracle import xsec_oracle as O
from paper_2510_20870_amd import synth

pytestmark = pytest.mark.gpu

N_LINES, N_GRID = 60_000, 200_000


@pytest.fixture(scope="module")
def data():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L = synth.make_lines(synth.ListSpec(N_LINES, 970.0, 1065.0, 92))
    return L, 1000.0 + 2e-4 * np.arange(N_GRID, dtype=np.float64)


def _opts(split=1, group=0):
    from paper_2510_20870_amd import xsec as X
    return X.Context.opts(X.XS_CUT_FIXED, 25.0, split=split, pts_per_lane=1, tile_group=group)


def _line_by_line_bytes(L, grid, pts, split, host):
    """Bytes a context holds after the call by the tile kernel alone, and its result."""
    import torch
    from paper_2510_20870_amd import xsec as X
    with X.Context(0) as c:
        h, g = c.load_lines(L, 16.0), c.set_grid(grid)
        o = _opts(split, 1)
        out = None if host else torch.empty((len(pts), len(grid)), dtype=torch.float64,
                                            device="cuda")
        sig = c.compute(h, g, pts, o, out=out, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        return c.memory_used()[0], sig if host else out.cpu().numpy()


# a point's records are 1.9 MB, its moments 0.9 MB, a row of the output or a partial 1.6 MB
@pytest.mark.parametrize("split,host", [(1, False), (1, True), (2, False), (2, True)])
def test_fits_line_by_line(data, split, host):
    import torch
    from paper_2510_20870_amd import xsec as X
    L, grid = data
    pts = [(0.01, 900.0)]
    need, want = _line_by_line_bytes(L, grid, pts, split, host)
    with X.Context(0, hbm_budget_bytes=need + 200_000) as c:
        h, g = c.load_lines(L, 16.0), c.set_grid(grid)
        for _ in range(2):   # the second beside what the first left
            out = None if host else torch.empty((1, N_GRID), dtype=torch.float64, device="cuda")
            sig = c.compute(h, g, pts, _opts(split), out=out,
                            stream=torch.cuda.current_stream())
            torch.cuda.synchronize()
            sig = sig if host else out.cpu().numpy()
            st = O.compare(sig[0], want[0], rel_tol=4e-6)   # both within 2e-6
            assert st["violations"] == 0, st
        assert int(c.count_evals(h, g, pts, _opts())[0]) > 0


def test_earlier_moments_do_not_block(data):
    """After a call by moments, everything that fits beside the line-by-line call's scratch."""
    from paper_2510_20870_amd import xsec as X
    L, grid = data
    pts = [(0.01, 900.0)]
    need, _ = _line_by_line_bytes(L, grid, pts, 1, True)
    with X.Context(0, hbm_budget_bytes=need + 3_500_000) as c:
        h, g = c.load_lines(L, 16.0), c.set_grid(grid)
        a = c.compute(h, g, pts, _opts())
        # selection takes no moments; its partials are 3.2 MB
        o = _opts(2)
        o.select_eps = 1e-4
        s = c.compute(h, g, pts, o)
        assert np.all(np.abs(s - a) <= 1.1e-4 * a)


@pytest.mark.parametrize("what", ["lines", "grid", "graph", "regrid", "server", "voigt"])
def test_scratch_is_given_back(data, what):
    """What needs device memory of its own fits beside the lists, grids and graphs in use: the
    scratch that finished calls hold gives way to it."""
    import torch
    from paper_2510_20870_amd import xsec as X
    L, grid = data
    pts = [(0.01, 900.0)]
    out = torch.empty((1, N_GRID), dtype=torch.float64, device="cuda")
    # lists and grid 3.2 MB, the call's records and moments 2.7 MB, 1 MB left
    with X.Context(0, hbm_budget_bytes=7_000_000) as c:
        h, g = c.load_lines(L, 16.0), c.set_grid(grid)
        c.compute(h, g, pts, _opts(), out=out, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        want = out.cpu().numpy()
        used, budget = c.memory_used()
        assert budget - used < 1_500_000
        if what == "lines":
            c.unload_lines(c.load_lines(L, 16.0))
        elif what == "grid":
            c.free_grid(c.set_grid(grid))
        elif what == "graph":
            gr = c.graph_create(h, g, pts, _opts(), out)
            out.fill_(-1.0)
            gr.launch(torch.cuda.current_stream())
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
            gr.close()
        elif what == "regrid":
            gd = c.set_grid(1000.0 + 4e-3 * np.arange(1000, dtype=np.float64))
            assert np.all(c.regrid(g, gd, want) > 0.0)
        elif what == "server":
            c.serve_start(mem_bytes=2_500_000)
        else:
            x = np.linspace(0.0, 10.0, 80_000)
            assert np.all(c.eval_voigt(x, np.full_like(x, 0.5)) > 0.0)
        if what != "server":   # (the arena keeps the memory)
            c.compute(h, g, pts, _opts(), out=out, stream=torch.cuda.current_stream())
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
