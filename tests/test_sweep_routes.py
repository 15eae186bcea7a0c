"""Which kernel a sweep runs in (slmpp_sweep_route), at both sides of each line
of the rule, and, on the GPU, the sweeps at those sizes against the FP64
oracle: persistent run-time tiles (3), persistent compile-time tiles (2) and
one tile per workgroup with compile-time (1) or run-time (0) segments.

Bounds as for the other single sweeps: 1e-13 of max |f| in FP64 storage, 64
FP32 ulp of it in FP32 (three stages each for TVD-RK)."""
import numpy as np
import pytest

import oracle as O
from paper_1702_08521_amd import slmpp as S
from paper_1702_08521_amd import workloads as W

# (nx, nv, storage, limiter, time, {axis: route})
CASES = [
    # run-time lengths, TVD-RK and other limiters at strides of 17 to 48 pencils
    # whose blocks need more threads than a workgroup has, and just above
    ([5, 7], [64, 40], 0, W.LIM_MPP, "rk3", {2: 3, 3: 3}),
    ([3, 4], [96, 44], 1, W.LIM_MPP, "rk3", {2: 3}),
    ([6, 6], [64, 36], 0, W.LIM_MPP, "rk3", {2: 3}),
    ([4, 5], [96, 44], 0, W.LIM_MP, "sl", {2: 3}),
    ([8, 8], [64, 40], 1, W.LIM_NONE, "sl", {2: 3}),
    ([3, 3], [128, 17], 0, W.LIM_MP, "sl", {2: 3}),
    ([3, 3], [128, 49], 0, W.LIM_MP, "sl", {2: 3}),
    ([2, 2], [500, 46], 0, W.LIM_NONE, "sl", {2: 3}),
    ([128], [40], 0, W.LIM_MP, "sl", {0: 3}),
    ([256], [44], 1, W.LIM_MP, "sl", {0: 3}),
    # rows that would be narrower than 64 bytes, and rows of whole 64-byte pieces
    ([5, 5], [384, 64], 1, W.LIM_MP, "sl", {2: 3}),
    ([9, 50], [60, 32], 1, W.LIM_MP, "sl", {1: 3, 2: 3}),
    # no tile of the run-time kernel: compile-time segments, or run-time ones
    ([40], [1200], 0, W.LIM_MPP, "rk3", {1: 1}),
    ([17], [3072], 0, W.LIM_MPP, "sl", {1: 1}),
    ([5], [3001], 0, W.LIM_MPP, "sl", {1: 0}),
    # compile-time tiles: small grids, half wavefronts, wide tiles
    ([11, 11], [64, 64], 0, W.LIM_MPP, "sl", {2: 3, 3: 3}),
    ([12, 11], [64, 64], 0, W.LIM_MPP, "sl", {2: 2, 3: 2}),
    ([8, 8], [64, 64], 1, W.LIM_MPP, "sl", {2: 3, 3: 3}),
    ([9, 9], [64, 64], 1, W.LIM_MPP, "sl", {2: 2, 3: 3}),
    ([35, 35], [16, 32], 0, W.LIM_MPP, "sl", {2: 3}),
    ([35, 35], [16, 32], 1, W.LIM_MPP, "sl", {2: 2}),
    ([35, 35], [24, 32], 0, W.LIM_MPP, "sl", {2: 2}),
    ([13, 60], [24, 30], 0, W.LIM_MPP, "sl", {1: 2}),
    ([13, 72], [24, 30], 0, W.LIM_MPP, "sl", {1: 3}),
    # blocks of more than 48 pencils that fill five wavefronts
    ([13, 13], [40, 64], 1, W.LIM_MP, "sl", {2: 3}),
    # one tile per workgroup: from 2^20 cells, blocks of five wavefronts, FP64 x
    # sweeps, long pencils, FP32 x sweeps up to 2^22 cells
    ([22, 24], [48, 44], 0, W.LIM_MPP, "sl", {2: 1}),
    ([20, 24], [48, 44], 0, W.LIM_MPP, "sl", {2: 3}),
    ([9, 128], [30, 31], 0, W.LIM_MPP, "sl", {1: 1}),
    ([8, 128], [30, 31], 0, W.LIM_MPP, "sl", {1: 3}),
    ([24, 48], [30, 31], 1, W.LIM_MPP, "sl", {1: 1}),
    ([50, 24], [30, 31], 0, W.LIM_MPP, "sl", {1: 3}),
    ([100, 24], [20, 25], 0, W.LIM_MPP, "sl", {1: 1}),
    ([3, 3], [384, 320], 1, W.LIM_MPP, "sl", {2: 1}),
    ([3, 3], [384, 300], 1, W.LIM_MPP, "sl", {2: 3}),
]
BIG = [
    ([97, 48], [30, 31], 1, W.LIM_MPP, "sl", {1: 3}),
    ([36, 128], [30, 31], 0, W.LIM_MPP, "sl", {1: 1}),
    ([74, 74], [1, 3072], 0, W.LIM_MPP, "sl", {3: 1}),
    ([73, 74], [1, 768], 0, W.LIM_MPP, "sl", {3: 3}),
    ([36, 36], [24, 2160], 1, W.LIM_MPP, "sl", {2: 3}),
    ([32, 36], [24, 2160], 1, W.LIM_MPP, "sl", {2: 2}),
    ([36, 36], [24, 336], 1, W.LIM_MPP, "sl", {2: 2}),
]


def _spec(case, order):
    nx, nv, _, limiter, time, _ = case
    D = len(nx)
    return W.spec(D, nx, nv, 0.0, 1.0, [-2.0 + 0.1 * l for l in range(D)], 2.5, order=order, limiter=limiter,
                  time=time)


def _dt(case, axis):
    return 0.44 / case[0][axis] / 2.5 if axis < len(case[0]) else 0.1


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", CASES + BIG, ids=lambda c: f"{c[0]}x{c[1]}-{c[2]}-{c[3]}-{c[4]}")
def test_route(case, order):
    desc = S.make_desc(_spec(case, order), case[2])
    for axis, route in case[5].items():
        assert S.sweep_route(desc, axis, _dt(case, axis)) == route, axis


def test_route_takes_every_stride_and_rejects_bad_arguments():
    """Pencils of up to 48 cells at any stride up to 200, and of any length up
    to 1024 next to blocks of up to 96 pencils, have a tile of the run-time
    kernel in every limiter and time integration."""
    for storage in (0, 1):
        for limiter, time in ((W.LIM_MP, "sl"), (W.LIM_NONE, "sl"), (W.LIM_MPP, "rk3")):
            for n, strides in [(k, range(2, 201)) for k in (5, 16, 31, 48)] + [
                    (k, range(2, 97)) for k in (60, 64, 96, 100, 128, 200, 256, 400, 512, 1000)]:
                for s in strides:
                    desc = S.make_desc(W.spec(2, [3, 3], [n, s], 0.0, 1.0, -1.0, 1.0, limiter=limiter, time=time),
                                       storage)
                    assert S.sweep_route(desc, 2) == 3, (n, s, storage, limiter, time)
    desc = S.make_desc(_spec(CASES[0], 5), 0)
    assert S.sweep_route(desc, 4) == S.sweep_route(desc, -1) == S.sweep_route(desc, 0, float("nan")) == -1
    desc.order = 6
    assert S.sweep_route(desc, 0) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("ci", range(len(CASES)))
def test_sweeps_of_each_route(ci):
    import torch

    case = CASES[ci]
    nx, nv, storage, limiter, time, axes = case
    D, nxs = len(nx), int(np.prod(nx))
    for order in (5, 7):
        spec = _spec(case, order)
        grid = O.make_grid(spec)
        f0 = W.random_field(grid.shape, 70 + ci)
        if storage:
            f0 = f0.astype(np.float32).astype(np.float64)
        ctx = S.Context(S.make_desc(spec, storage))
        for axis in axes:
            print(f"case nx={nx} nv={nv} storage={storage} lim={limiter} {time} order={order} axis={axis}", flush=True)
            ctx.init_f_host(f0)
            ref = f0.copy()
            dt = _dt(case, axis)
            if axis < D:
                ctx.advect_x(axis, dt)
                O.advect_x(grid, ref, axis, dt)
            else:
                l = axis - D
                h = (spec["v_hi"][l] - spec["v_lo"][l]) / nv[l]
                acc = W.random_accel(nxs, 1, 7 + axis, (0.44 if time == "rk3" else 2.6) * h / dt)
                ctx.advect_v(l, dt, torch.tensor(acc, dtype=torch.float64, device="cuda"))
                O.advect_v(grid, ref, l, dt, acc)
            err = np.abs(ctx.get_f() - ref).max() / np.abs(f0).max()
            assert err <= (1e-13 if storage == 0 else 64 * 2.0 ** -24) * (3 if time == "rk3" else 1), err
        ctx.close()
