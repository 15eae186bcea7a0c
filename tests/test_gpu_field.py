"""The field solve and what the step builds on it, at the edges of its
kernels: the one-dimensional convolution (tiny, odd, even and the longest
lengths, and the first beyond it), transform lengths divisible by four, by two
and odd, single-cell axes, the isolated solve where the potential with its
halo is as long as the doubled axis and longer, and calls of several steps,
whose closing and opening kicks run as one sweep in one dimension."""
import numpy as np
import pytest

import oracle as O
from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08521_amd import slmpp

    slmpp.lib()
    return slmpp


SOLVES = [([1], 2), ([2], 4), ([3], 6), ([5], 6), ([64], 6), ([255], 4), ([1022], 2), ([1024], 6),
          ([1030], 6), ([30, 37], 6), ([64, 18], 4), ([1, 9], 2), ([7, 1], 6), ([257, 3], 6),
          ([5, 6, 7], 6), ([8, 12, 16], 2), ([9, 1, 10], 4), ([1, 4, 33], 6), ([34, 5, 3], 6)]
ISOLATED = [([6, 6, 6], 6), ([7, 6, 9], 4), ([12, 8, 6], 2), ([16, 20, 11], 6), ([6, 5, 8], 6)]


def _solve(S, nx, order, isolated):
    import torch

    D = len(nx)
    hi = [1.0 + 0.3 * l for l in range(D)]
    spec = W.spec(D, nx, [2] * D, [0.0] * D, hi, -1.0, 1.0, kappa=4 * np.pi if isolated else -1.0,
                  poisson_order=order, field_bc="isolated" if isolated else "periodic")
    grid = O.make_grid(spec)
    nxs = int(np.prod(nx))
    rho = 1.0 + np.random.default_rng(nxs + order).random(nxs)
    ctx = S.Context(S.make_desc(spec, 0))
    r = torch.tensor(rho, dtype=torch.float64, device="cuda")
    acc = torch.full((D * nxs,), float("nan"), dtype=torch.float64, device="cuda")
    phi = torch.full((nxs,), float("nan"), dtype=torch.float64, device="cuda")
    ctx.poisson_solve(r, acc, phi)
    ctx.sync()
    assert np.array_equal(r.cpu().numpy(), rho)
    ctx.close()
    po, ao = O.poisson_isolated(grid, rho) if isolated else O.poisson_solve(grid, rho)
    # the angles of the roots of unity near 2 pi carry n roundings; a force is
    # a difference of potentials over 60 h / 110
    n = max(nx)
    tol = 32 * n * EPS * max(np.abs(po).max(), 1e-300)
    ep = np.abs(phi.cpu().numpy() - po).max()
    ea = [np.abs(acc.cpu().numpy()[l * nxs:(l + 1) * nxs] - ao[l * nxs:(l + 1) * nxs]).max() for l in range(D)]
    print(f"case solve nx={nx} order={order} isolated={isolated}: phi {ep:.2e} ({tol:.2e}) accel {ea}", flush=True)
    assert ep <= tol
    for l in range(D):
        assert ea[l] <= 2 * tol * 110.0 / (60.0 * hi[l] / nx[l])


@pytest.mark.parametrize("i", range(len(SOLVES)))
def test_periodic_solve(S, i):
    _solve(S, *SOLVES[i], False)


@pytest.mark.parametrize("i", range(len(ISOLATED)))
def test_isolated_solve(S, i):
    _solve(S, *ISOLATED[i], True)


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("nx,nv,order,v_bc", [(64, 128, 5, 1), (33, 47, 7, 1), (50, 34, 5, 0), (3, 600, 7, 1),
                                             (1100, 20, 5, 1)])
def test_steps_of_one_call_equal_single_calls(S, nx, nv, order, v_bc, storage):
    """The same kicks, sweeps and fields in the same order: bit for bit."""
    spec = W.landau_run(1, nx, nv, 0.5, 0.3, order)
    spec["v_bc"] = v_bc
    spec["kappa"] = -3.0
    s, gv = W.separable_factors(spec)
    out = []
    for calls in ([4], [1, 1, 1, 1]):
        ctx = S.Context(S.make_desc(spec, storage))
        ctx.init_f_separable(s, gv)
        for n in calls:
            ctx.step(2.0 * spec["dt"], n)
        out.append((ctx.get_f(), *ctx.get_field()))
        ctx.close()
    print(f"case steps {nx} x {nv} order={order} v_bc={v_bc} storage={storage}", flush=True)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    run = O.Run(spec, None if storage == 0 else O.init_separable(O.make_grid(spec), s, gv)
                .astype(np.float32).astype(np.float64))
    run.step(2.0 * spec["dt"], 4)
    assert np.abs(out[0][0] - run.f).sum() / run.f.sum() <= (1e-12 if storage == 0 else 1e-5)


def test_zero_time_step_keeps_f_and_leaves_the_field(S):
    spec = W.landau_run(2, 6, 12, 0.5, 0.3, 5)
    s, gv = W.separable_factors(spec)
    ctx = S.Context(S.make_desc(spec, 0))
    ctx.init_f_separable(s, gv)
    f0 = ctx.get_f()
    ctx.step(0.0, 2)
    rho, acc = ctx.get_field()
    print("case zero time step", flush=True)
    assert np.array_equal(ctx.get_f(), f0)
    grid = O.make_grid(spec)
    assert np.abs(rho - O.density_moment(grid, f0)).max() <= 64 * EPS * rho.max()
    assert np.abs(acc - O.field(grid, f0)).max() <= 1e-12 * np.abs(acc).max()
    ctx.close()


@pytest.mark.parametrize("time", ["sl", "rk3"])
@pytest.mark.parametrize("D", [1, 2])
def test_zero_time_step_runs_its_sweeps(S, D, time):
    """A step of no duration is its sweeps all the same: a cell that is no
    number makes the field, and with it every swept cell, no number; TVD-RK
    combines its stages in floating point (a few ulp of the oracle's)."""
    spec = dict(W.landau_run(D, 6, 16, 0.5, 0.3, 5), time=time)
    print(f"case zero time step D={D} time={time}", flush=True)
    f0 = W.random_field(spec["nx"][:D] + spec["nv"][:D], 3)
    ctx = S.Context(S.make_desc(spec, 0))
    ctx.init_f_host(f0)
    ctx.step(0.0, 2)
    f = ctx.get_f().reshape(f0.shape)
    assert np.abs(f - f0).max() <= (0.0 if time == "sl" else 64 * EPS * f0.max())
    f0.flat[5] = np.nan
    ctx.init_f_host(f0)
    ctx.step(0.0, 1)
    assert np.isnan(ctx.get_f()).all()
    ctx.close()
