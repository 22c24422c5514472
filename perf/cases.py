"""Cases for timing the public entry points over the range of work that users bring.

Every case is a dict of plain values. The inputs are seeded synthetic line lists with the
distributions of paper_2510_20870_amd/synth.py (centres uniform over the list's range, Einstein
A from 10^U(-6, 2), lower energies of mean 3000 cm^-1, gamma 0.03-0.1, n_T 0.4-0.8), at the
line densities of its workloads: 1e5 to 1e8 lines over 500-10000 cm^-1 (about 10 to 10500
lines per cm^-1), 8700 (the pressure-temperature table) and 33400 per cm^-1 (1e9 lines over
100-30000 cm^-1). Where such a list is too large to draw for every run, the case holds the
part of it that surrounds its grid, as a program that works window by window loads it.

Cross-sections of the FP32 path are stored as float32 (XS_F32), the type that its arithmetic
carries; those of the FP64 path as float64. A program keeps the line lists, grids, graphs and
output buffers, and one context with the shipped tuning cache; all of that is in prepare().
"""
import math
import os

import numpy as np
import torch

import paper_2510_20870_amd
from paper_2510_20870_amd import xsec

C2 = 6.62607015e-34 * 299792458.0 / 1.380649e-23 * 100.0
C_LIGHT = 299792458.0
AMU = 1.66053906660e-27
K_BOLTZ = 1.380649e-23
Q_A, Q_B, T_REF = 0.0343, 1.5, 296.0
WINDOW_MARGIN = 30.0      # lines kept on both sides of a window [cm^-1]
PARTNERS_J = 81


def _sigma(name, lines_per_cm, nu, width, points, **more):
    """A cross-section case: a window of `width` cm^-1 from `nu` on `points` grid points."""
    case = dict(name=name, kind="sigma", via="compute", lines_per_cm=float(lines_per_cm),
                nu=float(nu), width=float(width), points=int(points), spacing="uniform",
                list_lo=0.0, list_hi=0.0, npts=1, p_lo=0.1, p_hi=0.1, t_lo=1500.0, t_hi=1500.0,
                mass=16.0, cut=25.0, rule="fixed", precision="fp32", select_eps=0.0, tol=0.0,
                partners=False)
    case.update(more)
    return case


def listed():
    return [
        # the smallest call: 1e4 lines over 1000-1100 cm^-1 on 1e4 points, one (P, T); a
        # retrieval loop calls it over and over, so launches and latency count
        _sigma("small_point", 100, 1000.0, 100.0, 10000, list_lo=1000.0, list_hi=1100.0,
               p_lo=1.0, p_hi=1.0, t_lo=1000.0, t_hi=1000.0, mass=18.0, cut=10.0),
        # the same kind of small work captured once and replayed: three layers of an
        # atmosphere on a 10 cm^-1 window of the 1e5-line list
        _sigma("small_graph", 1e5 / 9500, 4000.0, 10.0, 1001, via="graph", list_lo=500.0,
               list_hi=10000.0, npts=3, p_lo=1e-3, p_hi=10.0, t_lo=500.0, t_hi=2000.0,
               mass=18.0),
        # an ordinary window of the 1e6-line list, odd size
        _sigma("window_1e6", 1e6 / 9500, 2100.0, 50.0, 5003, list_lo=500.0, list_hi=10000.0,
               p_lo=0.01, p_hi=0.01, t_lo=700.0, t_hi=700.0),
        # a window of the 1e8-line list: many lines per grid point, few grid points
        _sigma("window_1e8", 1e8 / 9500, 6000.0, 200.0, 20011, p_lo=0.3, p_hi=0.3,
               mass=44.0),
        # the mid-size single point: 1e7 lines over 500-10000 cm^-1 on the whole 0.01 cm^-1
        # grid (the largest case)
        _sigma("whole_1e7", 1e7 / 9500, 500.0, 9500.0, 950000, list_lo=500.0, list_hi=10000.0),
        # the 1e9-line list on its ln(nu) grid around 10000 cm^-1, low to high pressure, at
        # the loose error budget that the benchmark runs
        _sigma("slice_1e9", 1e9 / 29900, 10000.0, 200.0, 10413, spacing="ln", npts=3,
               p_lo=1e-4, p_hi=100.0, t_lo=500.0, t_hi=3000.0, tol=1e-5),
        # a pressure-temperature table with the FWHM cutoff and broadening partners
        _sigma("table_fwhm", 1e8 / 11500, 3000.0, 250.0, 25147, spacing="ln", npts=12,
               p_lo=1e-5, p_hi=100.0, t_lo=300.0, t_hi=3000.0, rule="fwhm", partners=True),
        # the FP64 path: a reference-grade point
        _sigma("point_fp64", 1e7 / 9500, 2000.0, 1000.0, 100003, precision="fp64"),
        # the FP64 path with main-contributor selection
        _sigma("select_fp64", 1e7 / 9500, 3000.0, 300.0, 30001, precision="fp64",
               select_eps=1e-4),
        # high pressure: every wing broad, two hot layers near 100 bar
        _sigma("high_pressure", 1e7 / 9500, 1500.0, 2000.0, 200000, npts=2, p_lo=30.0,
               p_hi=100.0, t_lo=800.0, t_hi=2500.0),
        # a burst of window requests through the server: lists of 1e5, 1e6 and 4e6 lines,
        # windows of 10 to 300 cm^-1, the results in device memory
        dict(name="serve_burst", kind="serve", requests=12, lists="100000,1000000,4000000",
             w_lo=10.0, w_hi=300.0, p_lo=1e-5, p_hi=100.0, t_lo=300.0, t_hi=3000.0),
        # computed rows resampled to bin means at a fixed resolving power, on the device
        dict(name="regrid_rows", kind="regrid", rows=12, points=600000, nu=500.0, width=9500.0,
             r_out=1000.0, mode="mean"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "slice", "table", "fp64", "select", "graph",
                       "serve", "regrid"])
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(3, 14), lists="100000,1000000,4000000",
                    w_lo=10.0, w_hi=round(_log(rng, 40.0, 300.0), 2), p_lo=1e-5, p_hi=100.0,
                    t_lo=300.0, t_hi=3000.0)
    if kind == "regrid":
        return dict(kind="regrid", rows=rng.randint(1, 12), points=int(_log(rng, 3e4, 6e5)),
                    nu=round(rng.uniform(300.0, 1000.0), 3), width=round(rng.uniform(2e3, 9e3), 3),
                    r_out=round(_log(rng, 100.0, 3e4), 1), mode=rng.choice(["mean", "linear"]))
    p_lo = _log(rng, 1e-5, 100.0)
    t_lo = rng.uniform(300.0, 3000.0)
    nu = rng.uniform(600.0, 9000.0)
    dens = _log(rng, 10.0, 33000.0)
    width = _log(rng, 10.0, 1500.0)
    more = dict(p_lo=p_lo, p_hi=p_lo, t_lo=t_lo, t_hi=t_lo, mass=rng.choice([16.0, 18.0, 28.0, 44.0]),
                cut=rng.choice([25.0, 25.0, 10.0]), tol=rng.choice([0.0, 0.0, 1e-5]))
    most = 2e10          # (line, point) pairs inside the cut
    if kind in ("slice", "table"):
        more.update(npts=rng.randint(2, 8), p_lo=1e-5, p_hi=100.0, t_lo=300.0, t_hi=3000.0)
    if kind == "slice":
        nu, dens, width = rng.uniform(600.0, 25000.0), _log(rng, 3000.0, 33000.0), _log(rng, 20.0, 200.0)
        more.update(spacing="ln", tol=1e-5)
    elif kind == "table":
        more.update(spacing="ln", rule="fwhm", cut=25.0, partners=rng.random() < 0.5)
        dens, width = _log(rng, 100.0, 9000.0), _log(rng, 20.0, 300.0)
    elif kind in ("fp64", "select"):
        more.update(precision="fp64", tol=0.0)
        most = 4e9
        if kind == "select":
            more.update(select_eps=rng.choice([1e-4, 1e-3]))
    elif kind == "graph":
        more.update(via="graph", npts=rng.randint(1, 4))
        width, most = _log(rng, 10.0, 60.0), 2e9
    # grid steps of 0.01 cm^-1, or of the ln(nu) grids (R about 3e5 to 5e5)
    step = 0.01 if more.get("spacing") != "ln" else nu * _log(rng, 1.9e-6, 3.2e-6)
    pairs = width / step * dens * 2 * more["cut"] * more.get("npts", 1)
    width *= min(1.0, most / pairs)
    if width < 3.0:      # a narrow window of a dense list: thin the list instead
        dens, width = dens * width / 3.0, 3.0
    points = max(65, int(width / step))
    case = _sigma("", dens, round(nu, 3), points * step, points, **more)
    del case["name"]
    return case


# ------------------------------------------------------------------------------ inputs
def _rng(seed, tag):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), tag])))


def _lines(n, lo, hi, seed, tag, partners=False):
    rng = _rng(seed, tag)
    gaps = np.cumsum(rng.standard_exponential(n + 1))
    nu0 = np.minimum(lo + (hi - lo) * (gaps[:n] / gaps[n]), np.nextafter(hi, lo))
    f = np.float32
    out = {"nu0": nu0,
           "A": np.power(f(10.0), rng.random(n, f) * f(8.0) - f(6.0)),
           "E_low": rng.standard_exponential(n, f) * f(3000.0),
           "gamma": rng.random(n, f) * f(0.07) + f(0.03),
           "n_T": rng.random(n, f) * f(0.4) + f(0.4),
           "g_up": rng.integers(1, 51, n, np.uint16)}
    if partners:
        out["J_low"] = np.rint(np.sqrt(out["E_low"] / f(10.0))).astype(np.uint16)
    return out


def _partners():
    """H2- and He-like broadening tables over the lower-state J."""
    J = np.arange(PARTNERS_J, dtype=np.float64)
    return {"vmr": np.array([0.85, 0.15]),
            "gamma": np.stack([0.09 / np.sqrt(1.0 + J / 15.0), 0.045 / np.sqrt(1.0 + J / 25.0)]),
            "n": np.stack([0.65 - 0.003 * J, 0.50 - 0.002 * J])}


def _span(case):
    """(first, last) wavenumber of the list that the program has loaded, and its lines."""
    lo, hi = case["list_lo"], case["list_hi"]
    if hi <= lo:
        lo, hi = case["nu"] - WINDOW_MARGIN, case["nu"] + case["width"] + WINDOW_MARGIN
    return lo, hi, max(1, int(round(case["lines_per_cm"] * (hi - lo))))


def _grid(case):
    n, nu, w = case["points"], case["nu"], case["width"]
    j = np.arange(n, dtype=np.float64)
    if case["spacing"] == "ln":
        return np.exp(math.log(nu) + j * (math.log((nu + w) / nu) / n))
    return nu + j * (w / n)


def _pts(case, seed):
    """(P, T) pairs: log-spaced pressures and linear temperatures, each moved by a few
    per cent with the seed."""
    rng, n = _rng(seed, 7), case["npts"]
    f = np.linspace(0.0, 1.0, n) if n > 1 else np.zeros(1)
    P = np.exp(np.log(case["p_lo"]) + f * np.log(case["p_hi"] / case["p_lo"]))
    T = case["t_lo"] + ((f * 3) % 1.0 if n > 3 else f) * (case["t_hi"] - case["t_lo"])
    return np.stack([P * rng.uniform(0.93, 1.07, n), T * rng.uniform(0.97, 1.03, n)], axis=1)


def _requests(case, seed):
    """(list, start, points, P, T) of a burst of requests: windows spread evenly in the
    logarithm of their width and over the lists, pressures too; where they lie, which
    pressure and what temperature each asks for follow the seed."""
    rng, out = _rng(seed, 9), []
    n, ids = case["requests"], len(case["lists"].split(","))
    layer = rng.permutation(n)
    for k in range(n):
        at = (k * 5) % n if n % 5 else k      # wide and narrow windows mixed
        w = case["w_lo"] * (case["w_hi"] / case["w_lo"]) ** ((at + 0.5) / n)
        P = case["p_lo"] * (case["p_hi"] / case["p_lo"]) ** ((layer[k] + rng.random()) / n)
        out.append((at % ids, float(rng.uniform(500.0, 10000.0 - w)), int(round(w / 0.01)), float(P),
                    float(rng.uniform(case["t_lo"], case["t_hi"]))))
    return out


_context = None
_serving = False


def _ctx():
    """The program's context, with the package's tuning cache."""
    global _context
    if _context is None:
        cache = os.path.join(os.path.dirname(paper_2510_20870_amd.__file__), "tune_cache.json")
        if os.path.exists(cache):
            xsec.tune_cache_load(cache)
        _context = xsec.Context(0)
    return _context


class State:
    """What a program holds between calls; its lists, grids and graphs are given back with it."""

    def __init__(self, case):
        self.case, self.ctx = case, _ctx()
        self.lines, self.grids, self.graph = [], [], None

    def __del__(self):
        if self.graph is not None:
            self.graph.close()
        for h in self.grids:
            self.ctx.free_grid(h)
        for h in self.lines:
            self.ctx.unload_lines(h)


def _opts(case):
    return xsec.Context.opts(
        xsec.XS_CUT_FIXED if case["rule"] == "fixed" else xsec.XS_CUT_MIN_FWHM, case["cut"], 100.0,
        xsec.XS_FP32_KAHAN if case["precision"] == "fp32" else xsec.XS_FP64,
        select_eps=case["select_eps"], tol=case["tol"],
        out_dtype=xsec.XS_F32 if case["precision"] == "fp32" else xsec.XS_F64)


def prepare(case, seed):
    global _serving
    s = State(case)
    if case["kind"] == "regrid":
        src = _grid(dict(case, spacing="ln"))
        dst = xsec.wavelength_grid(1e4 / (case["nu"] + case["width"]), 1e4 / case["nu"], case["r_out"])
        s.grids = [s.ctx.set_grid(src), s.ctx.set_grid(dst)]
        s.sigma = torch.from_numpy(_rows(case, seed)).cuda()
        s.out = torch.empty((case["rows"], len(dst)), dtype=torch.float64, device="cuda")
        return s
    if case["kind"] == "serve":
        if not _serving:
            s.ctx.serve_start(mem_bytes=8 << 30)
            _serving = True
        for k, n in enumerate(case["lists"].split(",")):
            s.lines.append(s.ctx.load_lines(_lines(int(n), 500.0, 10000.0, seed, 20 + k), (18.0, 16.0, 28.0)[k]))
        s.asked = _requests(case, seed)
        s.opts = xsec.Context.opts(xsec.XS_CUT_FIXED, 25.0, out_dtype=xsec.XS_F32)
        s.out = [torch.empty((1, n), dtype=torch.float32, device="cuda") for _, _, n, _, _ in s.asked]
        return s
    lo, hi, n = _span(case)
    s.lines = [s.ctx.load_lines(_lines(n, lo, hi, seed, 3, case["partners"]), case["mass"], q_a=Q_A, q_b=Q_B,
                                broadening=_partners() if case["partners"] else None)]
    s.grids = [s.ctx.set_grid(_grid(case))]
    s.pts, s.opts = _pts(case, seed), _opts(case)
    s.out = torch.empty((case["npts"], case["points"]), device="cuda",
                        dtype=torch.float32 if case["precision"] == "fp32" else torch.float64)
    if case["via"] == "graph":
        s.graph = s.ctx.graph_create(s.lines[0], s.grids[0], s.pts, s.opts, s.out)
    return s


def run(s):
    case = s.case
    if case["kind"] == "regrid":
        mode = xsec.XS_REGRID_BIN_MEAN if case["mode"] == "mean" else xsec.XS_REGRID_LINEAR
        return s.ctx.regrid(s.grids[0], s.grids[1], s.sigma, mode, out=s.out,
                            stream=torch.cuda.current_stream())
    if case["kind"] == "serve":
        waiting = [s.ctx.submit_window(s.lines[k], start, 0.01, n, [(P, T)], s.opts, out=o)
                   for (k, start, n, P, T), o in zip(s.asked, s.out)]
        for r in waiting:
            r.wait()
            r.release()
        return s.out
    if case["via"] == "graph":
        s.graph.launch(torch.cuda.current_stream())
        return s.out
    return s.ctx.compute(s.lines[0], s.grids[0], s.pts, s.opts, out=s.out,
                         stream=torch.cuda.current_stream())


def work(case):
    """Bytes: the lines that can reach the grid (26 bytes each), the grid and the output, once.
    Operations: each line's strength and widths at each (P, T) (about 100), and the Voigt
    function at the grid points in its core (within 8 Doppler widths, about 35 each); the
    smooth wings farther out can be summed for many lines at once."""
    if case["kind"] == "regrid":
        n = case["rows"] * case["points"]
        return {"bytes": 8 * (n + case["points"]) + 8 * (case["rows"] + 1) * case["r_out"] * 3, "flops": 3 * n}
    if case["kind"] == "serve":
        total = {"bytes": 0.0, "flops": 0.0}
        dens = [int(n) / 9500.0 for n in case["lists"].split(",")]
        for k in range(case["requests"]):
            w = case["w_lo"] * (case["w_hi"] / case["w_lo"]) ** ((k + 0.5) / case["requests"])
            lines = sum(dens) / len(dens) * (w + 50.0)
            core = 16 * 5000.0 * 4e-6 / 0.01
            total["bytes"] += 26 * lines + 4 * w / 0.01
            total["flops"] += lines * (100 + 35 * core)
        return total
    lo, hi, _ = _span(case)
    reach = min(hi, case["nu"] + case["width"] + case["cut"]) - max(lo, case["nu"] - case["cut"])
    lines, step = case["lines_per_cm"] * reach, case["width"] / case["points"]
    mid = case["nu"] + 0.5 * case["width"]
    b = mid / C_LIGHT * math.sqrt(2 * K_BOLTZ * 0.5 * (case["t_lo"] + case["t_hi"]) / (case["mass"] * AMU))
    core = min(16 * b, 2 * case["cut"]) / step
    out = 4 if case["precision"] == "fp32" else 8
    return {"bytes": 26 * lines + case["points"] * (8 + out * case["npts"]),
            "flops": case["npts"] * lines * (100 + 35 * core)}


# ------------------------------------------------------------------- values in 64 bits
def _rows(case, seed):
    """Smooth positive rows with narrow bumps, of the size of cross-sections."""
    rng, n = _rng(seed, 5), case["points"]
    x = np.arange(n, dtype=np.float64)
    base = 1e-22 * (1.5 + np.sin(x * rng.uniform(2e-4, 2e-3)))
    return np.stack([base * rng.random(n) ** 4 * 10.0 ** rng.uniform(-3, 1) for _ in range(case["rows"])])


def _faddeeva_core(x, y):
    """Re w(x + iy) for |z| <= 12: the trapezoidal rule on the Gaussian integral with step
    1/2, its nodes shifted away from x, and the residue of the pole where y < 2 pi."""
    h = 0.5
    shift = 0.5 * (torch.abs(x / h - torch.round(x / h)) < 0.25).to(x.dtype)
    s = torch.zeros_like(x)
    for n in range(-15, 15):
        t = (n + shift) * h
        s += torch.exp(-t * t) / ((x - t) ** 2 + y * y)
    s *= y * (h / math.pi)
    yc = torch.clamp(y, max=2 * math.pi)
    z = torch.complex(x, yc)
    p = 2.0 * torch.exp(-z * z) / (1.0 - torch.exp(-2j * math.pi * (z / h - shift)))
    return s + torch.where(y < 2 * math.pi, p.real, torch.zeros_like(s))


def _far(y2, r2, terms):
    """K sqrt(pi) / y from the asymptotic series of w."""
    u = 1.0 / r2
    t = 2.0 - 4.0 * (y2 * u)
    a = [1.0]
    for k in range(1, terms):
        a.append(a[-1] * (2 * k - 1) / 2.0)
    v0, v1 = torch.ones_like(u), t + 1.0
    total, up = torch.ones_like(u), u.clone()
    for k in range(1, terms):
        total += (a[k] * up) * v1
        if k + 1 < terms:
            v0, v1 = v1, t * v1 - v0
            up = up * u
    return u * total


def _params(L, P, T, mass, partners, rule, cut):
    """Line strengths, widths and cuts at one (P, T), on the GPU in 64 bits."""
    g = {k: torch.from_numpy(np.asarray(v, np.float64)).cuda() for k, v in L.items()}
    nu0, q = g["nu0"], Q_A * T ** Q_B
    S = (g["g_up"] * g["A"] / (8.0 * math.pi * C_LIGHT * 100.0 * nu0 * nu0) * torch.exp(-C2 * g["E_low"] / T)
         * -torch.expm1(-C2 * nu0 / T) / q)
    b = nu0 / C_LIGHT * math.sqrt(2.0 * K_BOLTZ * T / (mass * AMU))
    if partners is None:
        gam = g["gamma"] * P * torch.pow(torch.tensor(T_REF / T, dtype=torch.float64, device="cuda"), g["n_T"])
    else:
        j = torch.clamp(g["J_low"].long(), max=PARTNERS_J - 1)
        gam = 0.0
        for v, gt, nt in zip(partners["vmr"], partners["gamma"], partners["n"]):
            gam = gam + v * torch.from_numpy(gt * (T_REF / T) ** nt).cuda()[j]
        gam = gam * P
    if rule == "fixed":
        reach = torch.full_like(nu0, cut)
    else:
        f_l, f_g = 2.0 * gam, 2.0 * b * math.sqrt(math.log(2.0))
        reach = torch.clamp(100.0 * (0.5346 * f_l + torch.sqrt(0.2166 * f_l * f_l + f_g * f_g)), max=cut)
    return nu0, S, b, gam, reach


def _sum_profiles(nu0, S, b, gam, reach, grid):
    """sum_i S_i V_i over the lines inside their cuts, on every grid point."""
    ib, w = 1.0 / b, S / (b * math.sqrt(math.pi))
    y = gam * ib
    y2 = y * y
    wy = w * y / math.sqrt(math.pi)
    out = torch.zeros_like(grid)
    step = float(grid[-1] - grid[0]) / max(1, len(grid) - 1) if len(grid) > 1 else 1.0
    rows = int(min(1024, max(64, 24 * float(b.max()) / step)))
    cols = (1 << 22) // rows
    most = float(reach.max())
    host, grid_host = nu0.cpu().numpy(), grid.cpu().numpy()
    ib_min, y2_min = float(ib.min()), float(y2.min())
    for j0 in range(0, len(grid), rows):
        nu = grid[j0:j0 + rows]
        g0, g1 = grid_host[j0], grid_host[min(j0 + rows, len(grid)) - 1]
        lo, hi = np.searchsorted(host, [g0 - most * (1 + 1e-12), g1 + most * (1 + 1e-12)])
        for i0 in range(max(0, lo - 1), min(len(host), hi + 1), cols):
            i1 = min(len(host), hi + 1, i0 + cols)
            gap = max(0.0, host[i0] - g1, g0 - host[i1 - 1])
            d = nu[:, None] - nu0[None, i0:i1]
            inside = d.abs() <= reach[None, i0:i1]
            x = d * ib[None, i0:i1]
            yy2 = y2[None, i0:i1]
            r2 = x * x + yy2
            least = (gap * ib_min) ** 2 + y2_min
            if least > 1e4:
                k = _far(yy2, r2, 5)
            elif least > 144.0:
                k = _far(yy2, r2, 12)
            else:
                k = _far(yy2, torch.clamp(r2, min=144.0), 12)
                at = torch.nonzero(inside & (r2 < 144.0), as_tuple=True)
                for c in range(0, len(at[0]), 1 << 22):
                    r, q = at[0][c:c + (1 << 22)], at[1][c:c + (1 << 22)]
                    k[r, q] = _faddeeva_core(x[r, q], y[i0:i1][q]) * math.sqrt(math.pi) / y[i0:i1][q]
            out[j0:j0 + rows] += torch.where(inside, k * wy[None, i0:i1], 0.0).sum(dim=1)
    return out


def exact(case, seed):
    if case["kind"] == "regrid":
        src = _grid(dict(case, spacing="ln"))
        dst = xsec.wavelength_grid(1e4 / (case["nu"] + case["width"]), 1e4 / case["nu"], case["r_out"])
        rows = _rows(case, seed)
        if case["mode"] != "mean":
            return np.stack([np.interp(dst, src, y, left=0.0, right=0.0) for y in rows])
        mid = 0.5 * (dst[1:] + dst[:-1])
        edges = np.concatenate([[2 * dst[0] - mid[0]], mid, [2 * dst[-1] - mid[-1]]])
        a, b = np.maximum(edges[:-1], src[0]), np.minimum(edges[1:], src[-1])
        out = np.zeros((len(rows), len(dst)))
        # each bin: the trapezoids between its source nodes, and the partial ones at its ends
        i0 = np.searchsorted(src, a, side="right")
        i1 = np.maximum(i0, np.searchsorted(src, b, side="left"))
        many = i1 > i0
        first, last = np.minimum(i0, len(src) - 1), np.maximum(i1 - 1, 0)
        for r, y in enumerate(rows):
            ya, yb = np.interp(a, src, y), np.interp(b, src, y)
            piece = np.append(0.5 * (y[1:] + y[:-1]) * np.diff(src), 0.0)
            inner = np.add.reduceat(piece, np.stack([first, np.maximum(first, last)], 1).ravel())[::2]
            inner = np.where(last > first, inner, 0.0)
            ends = 0.5 * (ya + y[first]) * (src[first] - a) + 0.5 * (y[last] + yb) * (b - src[last])
            total = np.where(many, inner + ends, 0.5 * (ya + yb) * (b - a))
            out[r] = np.where(b > a, total / np.where(b > a, b - a, 1.0), 0.0)
        return out
    if case["kind"] == "serve":
        lists = [(_lines(int(n), 500.0, 10000.0, seed, 20 + k), (18.0, 16.0, 28.0)[k])
                 for k, n in enumerate(case["lists"].split(","))]
        out = []
        for k, start, n, P, T in _requests(case, seed):
            L, mass = lists[k]
            lo, hi = np.searchsorted(L["nu0"], [start - 26.0, start + 0.01 * n + 26.0])
            par = _params({f: v[lo:hi] for f, v in L.items()}, P, T, mass, None, "fixed", 25.0)
            grid = torch.from_numpy(start + np.arange(n, dtype=np.float64) * 0.01).cuda()
            out.append(_sum_profiles(*par, grid)[None, :])
        return out
    lo, hi, n = _span(case)
    L = _lines(n, lo, hi, seed, 3, case["partners"])
    grid = torch.from_numpy(_grid(case)).cuda()
    rows = []
    for P, T in _pts(case, seed):
        par = _params(L, float(P), float(T), case["mass"], _partners() if case["partners"] else None,
                      case["rule"], case["cut"])
        rows.append(_sum_profiles(*par, grid))
    return torch.stack(rows)
