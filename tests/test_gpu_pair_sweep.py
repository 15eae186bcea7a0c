"""The x_3 and x_2 sweeps of a step in one pass (pair_sweep_kernel): the
smallest and the largest spatial planes, planes that leave rounds and segments
uneven, velocity counts that end within a tile and that no vector divides,
both boundaries, and shifts up to several times around the pencil.

Without acceleration a step is its x sweeps alone: identical bit for bit to
slmpp_advect_x along x_3, x_2 and x_1.  With a field, against the FP64
oracle: 1e-12 (FP64 storage) or 1e-5 (FP32) in relative L1, as for the other
whole-step tests."""
import numpy as np
import pytest

import oracle as O
from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08521_amd import slmpp

    slmpp.lib()
    return slmpp


# (nx, nv, order, x_bc, largest shift in cells of x_3, taken in FP64, in FP32)
CASES = [
    ([3, 4, 4], [3, 5, 8], 5, 0, 0.4, True, True),       # smallest planes; 120 velocities
    ([2, 4, 3], [3, 5, 8], 5, 0, 0.4, False, False),     # below them
    ([2, 20, 24], [6, 7, 10], 7, 0, 1.4, True, True),    # 420 velocities: 13 tiles of 32 and 4
    ([2, 32, 32], [4, 6, 6], 5, 1, 0.5, True, False),    # largest in FP64, outflow
    ([2, 24, 24], [4, 6, 6], 5, 1, 0.5, True, True),     # largest in FP32, outflow
    ([2, 31, 33], [5, 4, 5], 7, 0, 40.0, True, False),   # 1023 rows, shifts around the pencil
    ([2, 32, 33], [4, 4, 4], 5, 0, 0.5, False, False),   # beyond the largest
    ([3, 5, 7], [3, 7, 12], 7, 1, 9.0, True, True),      # odd, shifts beyond an outflow pencil
    ([2, 4, 256], [2, 2, 14], 5, 0, 3.3, True, False),   # long x_3
    ([2, 4, 144], [2, 2, 14], 5, 1, 3.3, True, True),
    ([2, 143, 4], [2, 2, 14], 7, 0, 9.7, True, True),    # long x_2
    ([2, 13, 11], [3, 3, 3], 5, 0, 0.7, False, False),   # 27 velocities: no whole vectors
    ([2, 13, 11], [3, 5, 2], 5, 0, 0.7, True, False),    # 30: whole vectors in FP64
    ([1, 16, 17], [2, 3, 2], 7, 0, 2.6, True, True),     # 12 velocities: less than one tile
]


def _spec(nx, nv, order, x_bc):
    s = W.landau_run(3, nx[0], nv[0], 0.5, 0.3, order)
    s.update(nx=list(nx), nv=list(nv), x_bc=x_bc)
    return s


def _launches(ctx):
    t = ctx.timing_read()
    return sum(v["launches"] for k, v in t.items() if "sweep" in k or k == "kick_plane")


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("ci", range(len(CASES)))
def test_pair_pass(S, ci, storage):
    nx, nv, order, x_bc, most, *taken = CASES[ci]
    print(f"case nx={nx} nv={nv} order={order} x_bc={x_bc} shift={most} storage={storage}", flush=True)
    spec = dict(_spec(nx, nv, order, x_bc), kappa=0.0)
    f0 = W.random_field(nx + nv, 31 + ci)
    dt = most * (spec["x_hi"][2] - spec["x_lo"][2]) / nx[2] / 6.0
    ctx = S.Context(S.make_desc(spec, storage))
    ctx.init_f_host(f0)
    ctx.timing_enable(True)
    ctx.kick(dt)
    kick = _launches(ctx)
    ctx.init_f_host(f0)
    ctx.step(dt, 1)
    n_x = _launches(ctx) - 3 * kick
    assert n_x == (2 if taken[storage] else 3)
    a = ctx.get_f()
    ctx.init_f_host(f0)
    for axis in (2, 1, 0):
        ctx.advect_x(axis, dt)
    b = ctx.get_f()
    ctx.close()
    assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("ci", [0, 2, 4, 7])
def test_steps_with_the_pair_pass(S, ci, storage):
    nx, nv, order, x_bc = CASES[ci][:4]
    nv = [max(n, 8) for n in nv]
    print(f"case oracle nx={nx} nv={nv} order={order} x_bc={x_bc} storage={storage}", flush=True)
    spec = _spec(nx, nv, order, x_bc)
    ctx = S.Context(S.make_desc(spec, storage))
    sx, gv = W.separable_factors(spec)
    ctx.init_f_separable(sx, gv)
    ctx.step(spec["dt"], 3)
    got = ctx.get_f()
    ctx.close()
    f0 = O.init_separable(O.make_grid(spec), sx, gv)
    if storage:
        f0 = f0.astype(np.float32).astype(np.float64)
    run = O.Run(spec, f0)
    run.step(spec["dt"], 3)
    err = np.abs(got - run.f).sum() / np.abs(run.f).sum()
    assert err <= (1e-12 if storage == 0 else 1e-5), err
