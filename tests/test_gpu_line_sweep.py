"""Single sweeps at the edges of line_sweep_kernel's shapes against the FP64
oracle: row tiles that end within a block and within a vector, block tiles of
one and several blocks with odd lengths and a short last tile, the segment
lengths of small, middle and large grids (4, 8 and 16 cells in FP32), pencils
whose last segment is moved back, ghost regions wider than the pencil, shifts
beyond the ghost cells, both boundaries, every limiter, TVD-RK, and the row
sums of the x_1 sweep that end within a velocity block.

Bounds as for the other single sweeps: 1e-13 of max |f| in FP64 storage, 64
FP32 ulp of it in FP32 (three stages each for TVD-RK)."""
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


# (nx, nv, axes swept, largest shift in cells)
CASES = [
    ([3], [2047], (0, 1), 2.6),           # longest pencils in one tile each; 3-cell pencils
    ([1023], [50], (0, 1), 9.4),          # blocks of 50 pencils beside the 48 of a small block
    ([130], [4099 - 4], (1,), 0.4),       # beyond the kernel's pencils
    ([33, 5], [13, 49], (0, 1, 2, 3), 1.3),
    ([7, 9], [125, 67], (0, 1, 2, 3), 5.7),      # 5e5 cells: segments of 8
    ([19, 2], [17, 1], (0, 2, 3), 0.4),
    ([5, 3, 7], [9, 25, 25], (0, 2, 3, 4, 5), 0.45),     # odd blocks: 25, 625, 5625
    ([12, 11, 13], [15, 14, 13], (0, 1, 2, 3, 4, 5), 1.4),  # 4.7e6 cells: segments of 16
    ([6, 10, 9], [31, 17, 18], (0, 3, 5), 0.4),
    ([2, 2, 40], [33, 33, 27], (2, 4), 4.2),
]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("ci", range(len(CASES)))
def test_line_sweeps(S, ci, storage):
    import torch

    nx, nv, axes, most = CASES[ci]
    D = len(nx)
    for k, (order, limiter, x_bc, v_bc, rk) in enumerate([
            (7, W.LIM_MPP, 0, 1, False), (5, W.LIM_MP, 1, 0, False), (5, W.LIM_MPP, 0, 0, True),
            (7, W.LIM_NONE, 1, 1, False)]):
        if np.prod(nx) * np.prod(nv) > 2e6 and k > 1:
            continue
        spec = W.spec(D, nx, nv, 0.0, 1.0, [-2.0 + 0.1 * l for l in range(D)], 2.5, order=order,
                      limiter=limiter, x_bc=x_bc, v_bc=v_bc, time="rk3" if rk else "sl")
        grid = O.make_grid(spec)
        f0 = W.random_field(grid.shape, 50 * ci + k)
        if storage:
            f0 = f0.astype(np.float32).astype(np.float64)
        nxs = int(np.prod(nx))
        ctx = S.Context(S.make_desc(spec, storage))
        for axis in axes:
            print(f"case nx={nx} nv={nv} storage={storage} order={order} lim={limiter} bc=({x_bc},{v_bc}) "
                  f"rk={rk} axis={axis}", flush=True)
            shift = 0.44 if rk else most
            ctx.init_f_host(f0)
            ref = f0.copy()
            if axis < D:
                dt = shift * (1.0 / nx[axis]) / 2.5
                ctx.advect_x(axis, dt)
                O.advect_x(grid, ref, axis, dt)
            else:
                l = axis - D
                h = (spec["v_hi"][l] - spec["v_lo"][l]) / nv[l]
                acc = W.random_accel(nxs, 1, 7 + axis, shift * h / 0.1)
                ctx.advect_v(l, 0.1, torch.tensor(acc, dtype=torch.float64, device="cuda"))
                O.advect_v(grid, ref, l, 0.1, acc)
            err = np.abs(ctx.get_f() - ref).max() / np.abs(f0).max()
            assert err <= (1e-13 if storage == 0 else 64 * 2.0 ** -24) * (3 if rk else 1), err
        ctx.close()


@pytest.mark.parametrize("storage", [0, 1])
def test_row_sums_of_ragged_velocity_blocks(S, storage):
    """Steps of a grid large enough for the fused moment whose velocity
    blocks no tile divides: the density after the step against the moment of
    the f it left (before the closing kick, which keeps every cell's
    density up to the outflow at |v| = 6) and against the oracle's."""
    spec = W.landau_run(2, 40, 50, 0.5, 0.2, 5)
    spec["nv"] = [50, 53, 1]
    s, gv = W.separable_factors(spec)
    ctx = S.Context(S.make_desc(spec, storage))
    ctx.init_f_separable(s, gv)
    ctx.timing_enable(True)
    ctx.step(spec["dt"], 2)
    assert ctx.timing_read()["sweep_x1_moment"]["launches"] == 2
    rho, acc = ctx.get_field()
    f0 = O.init_separable(O.make_grid(spec), s, gv)
    if storage:
        f0 = f0.astype(np.float32).astype(np.float64)
    run = O.Run(spec, f0)
    run.step(spec["dt"], 2)
    ref = O.density_moment(run.grid, run.f)
    err = np.abs(rho - ref).max() / np.abs(ref).max()
    erra = np.abs(acc - run.accel).max() / np.abs(run.accel).max()
    print(f"case ragged row sums storage={storage}: rho {err:.2e} accel {erra:.2e}", flush=True)
    # outflow at 6 sigma: below 1e-8 of the density
    assert err <= 1e-7 and erra <= (1e-10 if storage == 0 else 1e-5)
    f = ctx.get_f()
    assert np.abs(f - run.f).sum() / run.f.sum() <= (1e-12 if storage == 0 else 1e-5)
    ctx.close()
