"""Timed workloads of the library, through its public entry points.

A case is a dict of plain values.  ``prepare`` builds what a user's program
holds before the call (the context or batch, with f initialised on the GPU),
``run`` makes one call and returns what it leaves, ``exact`` the same outputs
in 64-bit torch / numpy written from the paper's formulas alone, and ``work``
the bytes and operations of one call.  Kinds of cases:

  step      slmpp_step: Strang steps of a Vlasov-Poisson run (the main path)
  advect    slmpp_advect_x and slmpp_advect_v along every axis (a user who
            drives the splitting, e.g. scheme tests with another limiter)
  moments   what a run writes out between steps: velocity moments, velocity
            distribution and diagnostics
  ensemble  one step of a batch of uneven independent runs
"""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import torch

# exact() gives None above this many cell updates (time)
EXACT_UPDATES = 5.0e9


def _ints(text):
    return [int(x) for x in text.split("x")]


def _prod(v):
    p = 1
    for x in v:
        p *= int(x)
    return p


def _step(name, nx, nv, order, dtype, *, limiter="mpp", time="sl", field="periodic", sign="electro",
          merged=False, cfl=0.5, steps=1):
    return {"name": name, "kind": "step", "nx": nx, "nv": nv, "order": order, "dtype": dtype,
            "limiter": limiter, "time": time, "field": field, "sign": sign, "merged": merged,
            "cfl": cfl, "steps": steps}


def listed():
    return [
        # linear Landau damping in 1D1V (Test-3), one step per call: the
        # smallest run anyone makes, bound by launches
        _step("landau_1d1v_64x128_f64", "64", "128", 5, "f64"),
        # nonlinear Landau / two-stream grid, large time step (integer
        # shifts), several steps between outputs
        _step("landau_1d1v_256x512_f32", "256", "512", 7, "f32", cfl=3.0, steps=8),
        # 2D2V on a grid chosen for the box, not for the machine: odd and
        # unequal axes
        _step("landau_2d2v_ragged_f32", "30x37", "54x61", 5, "f32"),
        # 2D2V in double with power-of-two axes and merged half-kicks
        _step("landau_2d2v_64_f64", "64x64", "64x64", 7, "f64", merged=True, cfl=0.2, steps=3),
        # gravitational (Jeans) run at 32^3 x 32^3 in double
        _step("jeans_3d3v_32_f64", "32x32x32", "32x32x32", 5, "f64", sign="gravity", cfl=0.2),
        # 3D Landau damping at 48^3 x 48^3 in single: the largest run
        _step("landau_3d3v_48_f32", "48x48x48", "48x48x48", 7, "f32", cfl=0.2),
        # 3D3V on an anisotropic box
        _step("landau_3d3v_ragged_f32", "18x20x24", "30x36x42", 7, "f32"),
        # spherical collapse (Test-4): isolated field, outflow in x and v
        _step("collapse_3d3v_32x24_f32", "32x32x32", "24x24x24", 5, "f32", field="isolated"),
        # the paper's comparison scheme: RK-MPP5 time integration
        _step("rk3_2d2v_48x40_f64", "48x48", "40x40", 5, "f64", time="rk3", cfl=0.4),
        # single sweeps without the positivity limiter (SL-MP7)
        {"name": "advect_mp_3d3v_24_f32", "kind": "advect", "nx": "24x24x24", "nv": "24x24x24",
         "order": 7, "dtype": "f32", "limiter": "mp", "cfl": 1.4},
        # 256 uneven runs of a parameter study, 32 of them 2D2V
        {"name": "ensemble_256_f32", "kind": "ensemble", "runs": 256, "two_d": 32, "layout": 1,
         "dtype": "f32"},
        # outputs of a 3D3V run
        {"name": "moments_3d3v_24x40_f32", "kind": "moments", "nx": "24x24x24", "nv": "40x40x40",
         "order": 5, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _axes(rng, D, lo, hi, most):
    """D axis lengths: equal, or each of its own; at most `most` in product."""
    while True:
        if rng.random() < 0.4:
            v = [_log_int(rng, lo, hi)] * D
        else:
            v = [_log_int(rng, lo, hi) for _ in range(D)]
        if rng.random() < 0.5:
            v = [max(lo, (n + 3) // 4 * 4) for n in v]
        if _prod(v) <= most:
            return v


def draw(rng):
    what = rng.choices(["step", "rk3", "isolated", "advect", "moments", "ensemble"],
                       [56, 8, 8, 12, 10, 6])[0]
    dtype = rng.choice(["f32", "f64"])
    order = rng.choice([5, 7])
    if what == "ensemble":
        return {"kind": "ensemble", "runs": _log_int(rng, 8, 256), "two_d": rng.randint(0, 24),
                "layout": rng.randint(2, 10 ** 6), "dtype": dtype}
    D = 3 if what == "isolated" else rng.choice([1, 2, 3])
    if D == 1:
        nx = [_log_int(rng, 16, 1024)]
        # (RK needs |a dt / dv| <= 1: no much finer velocity than space grid)
        nv = [_log_int(rng, 24, 1024 if what != "rk3" else 4 * nx[0])]
    elif D == 2:
        nx, nv = _axes(rng, 2, 8, 64, 4096), _axes(rng, 2, 16, 96, 9216)
    else:
        nx, nv = _axes(rng, 3, 6, 32, 12000), _axes(rng, 3, 8, 44, 50000)
    case = {"kind": "step", "nx": "x".join(map(str, nx)), "nv": "x".join(map(str, nv)),
            "order": order, "dtype": dtype}
    if what == "moments":
        return {**case, "kind": "moments"}
    if what == "advect":
        return {**case, "kind": "advect", "limiter": rng.choice(["none", "mp", "mpp", "mpp"]),
                "cfl": rng.choice([0.4, 1.4, 3.0])}
    rk = what == "rk3"
    return {**case, "limiter": "mpp", "time": "rk3" if rk else "sl",
            "field": "isolated" if what == "isolated" else "periodic",
            "sign": "electro" if rk else rng.choice(["electro", "electro", "gravity"]),
            "merged": rng.random() < 0.25, "cfl": 0.4 if rk else rng.choice([0.2, 0.5, 0.5, 1.5, 3.0]),
            "steps": rng.choice([1, 1, 2, 4])}


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
LIMITERS = {"none": 0, "mp": 1, "mpp": 2}
VMAX = 6.0


def _centres(lo, hi, n):
    return lo + (np.arange(n, dtype=np.float64) + 0.5) * ((hi - lo) / n)


def _spec(case, rng):
    """Grid description (the keys of slmpp.make_desc), dt and the initial
    condition's factors s(x), g_l(v_l)."""
    nx, nv = _ints(case["nx"]), _ints(case["nv"])
    D = len(nx)
    isolated = case.get("field") == "isolated"
    gravity = isolated or case.get("sign") == "gravity"
    if isolated:
        x_lo, x_hi, vmax = -3.0, 3.0, 3.0
    elif gravity:
        x_lo, x_hi, vmax = 0.0, 1.0, 5.0
    else:
        x_lo, x_hi, vmax = 0.0, 4.0 * math.pi, VMAX
    spec = {"D": D, "nx": nx + [1] * (3 - D), "nv": nv + [1] * (3 - D),
            "x_lo": [x_lo] * 3, "x_hi": [x_hi] * 3, "v_lo": [-vmax] * 3, "v_hi": [vmax] * 3,
            "order": case["order"], "limiter": LIMITERS[case.get("limiter", "mpp")], "alpha": 4.0,
            "kappa": 4.0 * math.pi if gravity else -1.0, "poisson_order": 6,
            "x_bc": 1 if isolated else 0, "v_bc": 1, "time": case.get("time", "sl"),
            "merge_kicks": bool(case.get("merged", False)),
            "field_bc": "isolated" if isolated else "periodic"}
    xs = np.meshgrid(*[_centres(x_lo, x_hi, n) for n in nx], indexing="ij")
    if isolated:  # uniform sphere, slightly off centre
        off = rng.uniform(-0.05, 0.05, size=D)
        r2 = sum((x - o) ** 2 for x, o in zip(xs, off))
        s = np.where(r2 < 4.0, 3.0 / (32.0 * math.pi), 0.0)
        sigma = math.sqrt(0.05) * rng.uniform(0.95, 1.05)
        drift = [0.0] * D
    else:
        amp = rng.uniform(0.01, 0.1) if not gravity else rng.uniform(0.005, 0.02)
        k = 2.0 * math.pi / (x_hi - x_lo)
        s = 1.0 + amp * sum(np.cos(k * x + rng.uniform(0.0, 2.0 * math.pi)) for x in xs)
        if gravity:  # wave number half the Jeans one
            s = s * (2.0 * k) ** 2 / (4.0 * math.pi)
        sigma, drift = 1.0, rng.uniform(-0.1, 0.1, size=D)
    gs = []
    for n, u in zip(nv, drift):
        v = _centres(-vmax, vmax, n) - u
        gs.append(np.exp(-v * v / (2.0 * sigma * sigma)) / (math.sqrt(2.0 * math.pi) * sigma))
    dt = case.get("cfl", 0.5) * min((x_hi - x_lo) / n for n in nx) / vmax
    return spec, dt, np.ascontiguousarray(s).ravel(), gs


def _case_rng(seed):
    return np.random.default_rng([170208521, int(seed)])


NX_1D = (32, 48, 64, 96, 128, 192, 256)
NV_1D = (64, 96, 128, 192, 256, 384, 512)


def _ensemble_runs(case):
    """Geometry of the runs (fixed by the case): cases of kind step."""
    r = np.random.default_rng([31, int(case["layout"])])
    n, two = int(case["runs"]), min(int(case["two_d"]), int(case["runs"]))
    runs = []
    for i in range(n):
        order = 5 if r.random() < 0.5 else 7
        if i >= n - two:
            nx, nv = "32x32", "64x64"
        else:
            nx, nv = str(int(r.choice(NX_1D))), str(int(r.choice(NV_1D)))
        runs.append({"nx": nx, "nv": nv, "order": order, "dtype": case["dtype"], "cfl": 0.5})
    return runs


def _accel(case, rng, nxs, D, dt):
    """Acceleration of the advect cases: fractional shifts and some of
    several cells (|a dt / h| up to about 2.5)."""
    nv = _ints(case["nv"])
    return [rng.uniform(-2.5, 2.5, size=nxs) * (2.0 * VMAX / nv[l]) / dt for l in range(D)]


def _es(case):
    return 8 if case["dtype"] == "f64" else 4


def _tdtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


# ----------------------------------------------------------------------------
# the framework's side
# ----------------------------------------------------------------------------
def prepare(case, seed):
    from paper_1702_08521_amd import slmpp

    storage = slmpp.F64 if case["dtype"] == "f64" else slmpp.F32
    rng = _case_rng(seed)
    if case["kind"] == "ensemble":
        specs = [_spec(c, rng) for c in _ensemble_runs(case)]
        shapes = [tuple(sp["nx"][:sp["D"]]) + tuple(sp["nv"][:sp["D"]]) for sp, _, _, _ in specs]
        sizes = [_prod(sh) for sh in shapes]
        # every run's f in one buffer, each at a multiple of 64 cells
        flat = torch.zeros(sum((n + 63) // 64 * 64 for n in sizes), dtype=_tdtype(case), device="cuda")
        fs, off = [], 0
        for n, sh in zip(sizes, shapes):
            fs.append(flat[off:off + n].view(sh))
            off += (n + 63) // 64 * 64
        b = slmpp.Batch([slmpp.make_desc(sp, storage) for sp, _, _, _ in specs],
                        [dt for _, dt, _, _ in specs], fs=fs)
        for i, (_, _, s, gs) in enumerate(specs):
            b.init_separable(i, s, gs)
        b.autotune()
        return {"kind": "ensemble", "batch": b, "f": flat}
    spec, dt, s, gs = _spec(case, rng)
    ctx = slmpp.Context(slmpp.make_desc(spec, storage))
    ctx.init_f_separable(s, gs)
    state = {"kind": case["kind"], "ctx": ctx, "dt": dt, "D": spec["D"]}
    nxs, nvs = ctx.nxs, ctx.ncell // ctx.nxs
    if case["kind"] == "step":
        state["steps"] = case["steps"]
    elif case["kind"] == "advect":
        state["accel"] = [torch.from_numpy(a).cuda() for a in _accel(case, rng, nxs, spec["D"], dt)]
    else:
        new = lambda n: torch.empty(n, dtype=torch.float64, device="cuda")  # noqa: E731
        state.update(rho=new(nxs), mean=new(spec["D"] * nxs), disp=new(spec["D"] * nxs), F=new(nvs))
    return state


def run(state):
    kind = state["kind"]
    if kind == "ensemble":
        state["batch"].step(1)
        return state["f"]
    ctx = state["ctx"]
    if kind == "step":
        ctx.step(state["dt"], state["steps"])
        # f whole, as a few slabs of x_1
        return list(ctx.f.split((ctx.f.shape[0] + 3) // 4))
    if kind == "advect":
        for l in range(state["D"]):
            ctx.advect_v(l, state["dt"], state["accel"][l])
        for l in range(state["D"]):
            ctx.advect_x(l, state["dt"])
        return ctx.f
    ctx.velocity_moments(state["rho"], state["mean"], state["disp"])
    ctx.velocity_distribution(state["F"])
    return state["rho"], state["mean"], state["disp"], state["F"], ctx.diag()


# floating-point operations of one cell update: the flux (2 order - 1), the
# MP constraint's early accept (about 8), the PP test (3) and the update (3)
def _update_flops(order):
    return 2 * order - 1 + 14


def _sweeps(case):
    D = len(_ints(case["nx"]))
    if case["kind"] == "advect":
        return 2 * D
    steps = case.get("steps", 1)
    n = steps * (2 * D if case.get("merged") else 3 * D) + (D if case.get("merged") else 0)
    return n * (3 if case.get("time") == "rk3" else 1)


def work(case):
    """Bytes: f read and written once by the call (outputs only: f read
    once, and the results).  Operations: those of the sweeps, or 2 per cell,
    moment and pass of the outputs."""
    if case["kind"] == "ensemble":
        cells = [(_prod(_ints(c["nx"])) * _prod(_ints(c["nv"])), c) for c in _ensemble_runs(case)]
        return {"bytes": 2.0 * _es(case) * sum(n for n, _ in cells),
                "flops": float(sum(n * 3 * len(_ints(c["nx"])) * _update_flops(c["order"]) for n, c in cells))}
    nxs, nvs, D = _prod(_ints(case["nx"])), _prod(_ints(case["nv"])), len(_ints(case["nx"]))
    cells = float(nxs) * nvs
    if case["kind"] == "moments":
        return {"bytes": cells * _es(case) + 8.0 * (nxs * (1 + 2 * D) + nvs),
                "flops": cells * (2 * (1 + 2 * D) + 4)}
    return {"bytes": 2.0 * cells * _es(case),
            "flops": cells * _sweeps(case) * _update_flops(case["order"])}


# ----------------------------------------------------------------------------
# the same in 64 bits, from the paper's formulas (torch, no library code)
# ----------------------------------------------------------------------------
def _flux_rows(order):
    """Coefficients c[k][j] of Phi_{i-1/2}(zeta) = sum_k (sum_j c[k][j]
    zeta^j) f_{i-h+k}: the mean over the last zeta of a cell left of the
    face of the degree order - 1 polynomial whose cell averages are the
    order cells around it (three, or four, upwind of the face)."""
    h = 3 if order == 5 else 4
    nodes = [Fraction(k - h) for k in range(order + 1)]  # faces; the flux face at 0
    rows = []
    for k in range(order):
        # primitive of the unit average in cell k: 0 up to face k, then 1;
        # Lagrange polynomial through the order + 1 faces
        poly = [Fraction(0)] * (order + 1)
        for m in range(k + 1, order + 1):
            p, den = [Fraction(1)], Fraction(1)
            for q in range(order + 1):
                if q != m:
                    p = [(p[i - 1] if i else 0) - nodes[q] * (p[i] if i < len(p) else 0)
                         for i in range(len(p) + 1)]
                    den *= nodes[m] - nodes[q]
            poly = [a + b / den for a, b in zip(poly, p)]
        # (P(0) - P(-zeta)) / zeta
        rows.append([float(-poly[j + 1] * (-1) ** (j + 1)) for j in range(order)])
    return rows


FLUX_ROWS = {5: _flux_rows(5), 7: _flux_rows(7)}


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))


def _median(a, b, c):
    return a + _minmod(b - a, c - a)


def _limited(phi, r, zeta, limiter, alpha):
    """MP constraint (App. A) and PP limiter of the fluxes leaving the cells
    r[2]; r: the five cells around the upwind cell."""
    fm2, fm1, f0, fp1, fp2 = r
    if limiter == 0:
        return phi
    dm1, d0, dp1 = fm2 - 2 * fm1 + f0, fm1 - 2 * f0 + fp1, f0 - 2 * fp1 + fp2
    fmp = f0 + _minmod(fp1 - f0, alpha * (f0 - fm1))
    m4 = lambda a, b: _minmod(_minmod(4 * a - b, 4 * b - a), _minmod(a, b))  # noqa: E731
    ful = f0 + alpha * (f0 - fm1)
    fmd = 0.5 * (f0 + fp1) - 0.5 * m4(d0, dp1)
    flc = f0 + 0.5 * (f0 - fm1) + 4.0 / 3.0 * m4(dm1, d0)
    lo = torch.maximum(torch.minimum(torch.minimum(f0, fp1), fmd), torch.minimum(torch.minimum(f0, ful), flc))
    hi = torch.minimum(torch.maximum(torch.maximum(f0, fp1), fmd), torch.maximum(torch.maximum(f0, ful), flc))
    phi = torch.where((phi - f0) * (phi - fmp) < 0, phi, _median(phi, lo, hi))
    if limiter == 1:
        return phi
    one = torch.ones_like(phi)

    def theta(u, up):
        den = up - u
        t = torch.where(den > 0, (up / torch.where(den > 0, den, one)).clamp(0.0, 1.0), torch.zeros_like(den))
        return torch.where(u < 0, t, one)

    th = torch.minimum(theta(f0 - 2 * zeta * phi, f0 - 2 * zeta * f0),
                       theta(fp1 + 2 * zeta * phi, fp1 + 2 * zeta * f0))
    return th * phi + (1 - th) * f0


def _pencils(g, xi, order, limiter, alpha, outflow, rk):
    """One sweep of the pencils g[p, :] by xi[p] cells."""
    n = g.shape[1]
    if rk:
        shift, zeta = torch.zeros_like(xi), xi
    else:
        shift = torch.floor(xi + 0.5)
        zeta = xi - shift
    back = zeta < 0
    z = zeta.abs()[:, None]
    m = torch.arange(-4, n + 4, device=g.device)
    cell = torch.where(back[:, None], n - 1 - m, m) - shift.long()[:, None]
    if outflow:
        r = torch.where((cell >= 0) & (cell < n), g.gather(1, cell.clamp(0, n - 1)), torch.zeros((), dtype=g.dtype, device=g.device))
    else:
        r = g.gather(1, cell % n)
    at = lambda k: r[:, 3 + k:3 + k + n + 1]  # cells m - 1 + 1 + k ..., upwind cells m = -1..n-1 at k = 0  # noqa: E731
    zw = torch.zeros_like(z) if rk else z
    phi = torch.zeros_like(at(0))
    lo = -2 if order == 5 else -3
    for k, row in enumerate(FLUX_ROWS[order]):
        w = torch.zeros_like(zw)
        for c in reversed(row):
            w = w * zw + c
        phi = phi + w * at(lo + k)
    phi = _limited(phi, [at(k) for k in (-2, -1, 0, 1, 2)], z, limiter, alpha)
    out = r[:, 4:4 + n] - z * (phi[:, 1:] - phi[:, :-1])
    return torch.where(back[:, None], out.flip(1), out)


def _sweep(f, shape, axis, xi_of, spec, outflow):
    """Sweep of f (64 bits, updated in place) along `axis`; xi_of(pencils):
    the offsets of the pencils with these numbers (outer * inner + j)."""
    n = shape[axis]
    inner = _prod(shape[axis + 1:])
    outer = _prod(shape[:axis])
    v = f.view(outer, n, inner)
    rk = spec["time"] == "rk3"
    go = lambda g, xi: _pencils(g, xi, spec["order"], spec["limiter"], spec["alpha"], outflow, rk)  # noqa: E731
    block = max(1, (1 << 22) // n)
    for o0 in range(0, outer, max(1, block // inner)):
        o1 = min(outer, o0 + max(1, block // inner))
        for j0 in range(0, inner, block):
            j1 = min(inner, j0 + block)
            g = v[o0:o1, :, j0:j1].transpose(1, 2).reshape(-1, n)
            p = (torch.arange(o0, o1, device=f.device)[:, None] * inner
                 + torch.arange(j0, j1, device=f.device)[None, :]).reshape(-1)
            xi = xi_of(p)
            u = go(g, xi)
            if rk:
                u = 0.75 * g + 0.25 * go(u, xi)
                u = (g + 2.0 * go(u, xi)) / 3.0
            v[o0:o1, :, j0:j1] = u.reshape(o1 - o0, j1 - j0, n).transpose(1, 2)


def _box_mean_inverse_r(h):
    """Mean of 1/r over a box centred at the origin (closed form)."""
    a, b, c = (0.5 * x for x in h)
    r = math.sqrt(a * a + b * b + c * c)
    v = 0.0
    for p, q, s in ((a, b, c), (b, c, a), (c, a, b)):
        v += q * s * math.asinh(p / math.hypot(q, s)) - 0.5 * p * p * math.atan(q * s / (p * r))
    return 8.0 * v / (h[0] * h[1] * h[2])


def _acceleration(rho, spec):
    """Components of -grad phi for the density rho[x] (64 bits)."""
    D = spec["D"]
    n = spec["nx"][:D]
    h = [(spec["x_hi"][l] - spec["x_lo"][l]) / n[l] for l in range(D)]
    dev = rho.device
    axes = list(range(D))
    if spec["field_bc"] == "isolated":
        m = [2 * k for k in n]
        sep = []
        for l in axes:
            i = torch.arange(m[l], device=dev, dtype=torch.float64)
            i = torch.where(i < n[l], i, i - m[l]) * h[l]
            sep.append(i.view([-1 if k == l else 1 for k in axes]))
        r2 = sum(s * s for s in sep)
        inv = torch.where(r2 > 0, 1.0 / torch.sqrt(torch.where(r2 > 0, r2, torch.ones_like(r2))),
                          torch.full_like(r2, _box_mean_inverse_r(h)))
        g = -spec["kappa"] / (4.0 * math.pi) * _prod_f(h) * inv
        pad = torch.zeros(m, dtype=torch.float64, device=dev)
        pad[tuple(slice(0, k) for k in n)] = rho
        phi = torch.fft.ifftn(torch.fft.fftn(pad) * torch.fft.fftn(g)).real
    else:
        sym = torch.zeros([1] * D, dtype=torch.float64, device=dev)
        for l in axes:
            th = 2.0 * math.pi * torch.arange(n[l], device=dev, dtype=torch.float64) / n[l]
            a, b, c = torch.sin(0.5 * th), torch.sin(th), torch.sin(1.5 * th)
            s = (-2 * c * c + 27 * b * b - 270 * a * a) / 45.0 / (h[l] * h[l])
            sym = sym + s.view([-1 if k == l else 1 for k in axes])
        sym[(0,) * D] = 1.0
        green = spec["kappa"] / sym
        green[(0,) * D] = 0.0
        phi = torch.fft.ifftn(torch.fft.fftn(rho) * green).real
    out = []
    for l in axes:
        P = lambda k: torch.roll(phi, -k, l)  # noqa: E731
        d = (45.0 * (P(1) - P(-1)) - 9.0 * (P(2) - P(-2)) + (P(3) - P(-3))) / (60.0 * h[l])
        out.append(-d[tuple(slice(0, k) for k in n)])
    return out


def _prod_f(v):
    p = 1.0
    for x in v:
        p *= x
    return p


class _Exact:
    """A run in 64 bits from the same initial data as the library's."""

    def __init__(self, spec, s, gs, dtype, device):
        self.spec, self.D = spec, spec["D"]
        D = self.D
        self.nx, self.nv = spec["nx"][:D], spec["nv"][:D]
        self.shape = list(self.nx) + list(self.nv)
        self.hx = [(spec["x_hi"][l] - spec["x_lo"][l]) / self.nx[l] for l in range(D)]
        self.hv = [(spec["v_hi"][l] - spec["v_lo"][l]) / self.nv[l] for l in range(D)]
        self.device = device
        f = torch.from_numpy(s).to(device).view(list(self.nx) + [1] * D)
        for l, g in enumerate(gs):
            f = f * torch.from_numpy(g).to(device).view([-1 if k == D + l else 1 for k in range(2 * D)])
        self.f = f.to(torch.float32).to(torch.float64) if dtype == "f32" else f.contiguous()

    def rho(self):
        nxs = _prod(self.nx)
        return self.f.view(nxs, -1).sum(1).view(self.nx) * _prod_f(self.hv)

    def advect_x(self, l, dt):
        sp = self.spec
        c = sp["v_lo"][l] + (torch.arange(self.nv[l], device=self.device, dtype=torch.float64) + 0.5) * self.hv[l]
        xi = c * dt / self.hx[l]
        inner = _prod(self.shape[l + 1:])
        div = _prod(self.shape[self.D + l + 1:])
        of = lambda p: xi[(p % inner) // div % self.nv[l]]  # noqa: E731
        _sweep(self.f, self.shape, l, of, sp, sp["x_bc"] == 1)

    def advect_v(self, l, dt, accel):
        sp = self.spec
        xi = accel.reshape(-1) * dt / self.hv[l]
        per = _prod(self.nv) // self.nv[l]  # pencils of a spatial cell
        _sweep(self.f, self.shape, self.D + l, lambda p: xi[p // per], sp, sp["v_bc"] == 1)

    def kick(self, dt):
        for l in range(self.D):
            self.advect_v(l, dt, self.a[l])

    def field(self):
        self.a = _acceleration(self.rho(), self.spec)

    def step(self, dt, steps):
        self.field()
        merged = self.spec["merge_kicks"]
        self.kick(0.5 * dt)
        for i in range(steps):
            for l in reversed(range(self.D)):
                self.advect_x(l, dt)
            self.field()
            last = i + 1 == steps
            self.kick(0.5 * dt if last or not merged else dt)
            if not last and not merged:
                self.kick(0.5 * dt)


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    rng = _case_rng(seed)
    if case["kind"] == "ensemble":
        runs = _ensemble_runs(case)
        parts = []
        for c in runs:
            spec, dt, s, gs = _spec(c, rng)
            e = _Exact(spec, s, gs, case["dtype"], dev)
            e.step(dt, 1)
            n = e.f.numel()
            parts += [e.f.reshape(-1), torch.zeros((-n) % 64, dtype=torch.float64, device=dev)]
        return torch.cat(parts)
    cells = float(_prod(_ints(case["nx"]))) * _prod(_ints(case["nv"]))
    if cells * (_sweeps(case) if case["kind"] != "moments" else 2) > EXACT_UPDATES:
        return None
    spec, dt, s, gs = _spec(case, rng)
    e = _Exact(spec, s, gs, case["dtype"], dev)
    if case["kind"] == "step":
        e.step(dt, case["steps"])
        return list(e.f.split((e.f.shape[0] + 3) // 4))
    D, nxs = e.D, _prod(e.nx)
    if case["kind"] == "advect":
        acc = [torch.from_numpy(a).to(dev) for a in _accel(case, rng, nxs, D, dt)]
        for l in range(D):
            e.advect_v(l, dt, acc[l])
        for l in range(D):
            e.advect_x(l, dt)
        return e.f
    rho = e.rho()
    tot = e.f.view(nxs, -1).sum(1)
    mean, disp = [], []
    for l in range(D):
        v = spec["v_lo"][l] + (torch.arange(e.nv[l], device=dev, dtype=torch.float64) + 0.5) * e.hv[l]
        m = e.f.view([nxs] + e.nv).sum(dim=[1 + k for k in range(D) if k != l]) if D > 1 else e.f.view(nxs, -1)
        u = (m * v).sum(1) / tot
        mean.append(u)
        disp.append((m * (v[None, :] - u[:, None]) ** 2).sum(1) / tot)
    F = e.f.view(nxs, -1).sum(0) * _prod_f(e.hx)
    a = _acceleration(rho, spec)
    ang = -2.0 * math.pi * torch.arange(e.nx[0], device=dev, dtype=torch.float64) / e.nx[0]
    a1 = a[0].reshape(e.nx[0], -1).sum(1)
    mode = math.hypot(float((a1 * torch.cos(ang)).sum()), float((a1 * torch.sin(ang)).sum())) / nxs
    diag = {"mass": float(rho.sum()) * _prod_f(e.hx), "f_min": float(e.f.min()), "f_max": float(e.f.max()),
            "field_energy": 0.5 * float(sum((x * x).sum() for x in a)) * _prod_f(e.hx),
            "mode_amp": mode, "nonfinite": int((~torch.isfinite(e.f)).sum())}
    return rho.reshape(-1), torch.cat(mean), torch.cat(disp), F, diag
