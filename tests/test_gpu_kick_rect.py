"""The two-axis kick pass on velocity planes of any size (kick_rect_kernel):
the smallest planes, rows and planes that are no whole number of vectors,
the largest planes that fit, sizes just beyond, the size rule of large grids,
merged kicks, and shifts beyond the ring of zero cells.

With the pass and with SLMPP_FLAG_SEPARATE_KICKS the results must be
identical bit for bit, and match the FP64 oracle to 1e-12 (FP64 storage) or
1e-5 (FP32) in relative L1, as for the square planes."""
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


# (nx, nv, order, kappa, merged kicks, taken in FP64, taken in FP32)
CASES = [
    ([5, 6], [8, 8], 5, -1.0, False, True, True),            # smallest
    ([5, 6], [9, 13], 7, -100.0, False, True, True),         # odd planes, whole wavefront idle
    ([4, 4], [7, 40], 7, -1.0, False, False, False),         # below the smallest
    ([8, 8], [32, 33], 7, -1.0, True, True, True),
    ([6, 5], [21, 13], 5, -100.0, True, True, True),
    ([4, 3], [80, 72], 5, -100.0, False, True, True),        # whole rows of vectors
    ([3, 3], [88, 88], 7, -1.0, False, False, True),         # LDS full in FP64
    ([3, 2], [256, 31], 5, -1.0, False, False, True),        # longest pencils
    ([3, 2], [31, 257], 5, -1.0, False, False, False),
    ([4, 3, 4], [8, 10, 15], 7, -1.0, False, True, True),
    ([3, 2, 2], [5, 36, 43], 5, -100.0, True, True, True),
    ([1, 3], [64, 11], 7, -1.0, False, True, True),
]


def _run(S, spec, storage, n, separate):
    ctx = S.Context(S.make_desc(dict(spec, separate_kicks=separate), storage))
    ctx.init_f_separable(*W.separable_factors(spec))
    ctx.timing_enable(True)
    ctx.step(spec["dt"], n)
    launches = ctx.timing_read()["kick_plane"]["launches"]
    f = ctx.get_f()
    ctx.close()
    return f, launches


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("ci", range(len(CASES)))
def test_rect_pass(S, ci, storage):
    nx, nv, order, kappa, merge, *taken = CASES[ci]
    D, n = len(nx), 3
    print(f"case nx={nx} nv={nv} order={order} kappa={kappa} merge={merge} storage={storage}", flush=True)
    spec = W.landau_run(D, nx[0], nv[-1], 0.5, 0.3, order)
    spec.update(nx=nx + [1] * (3 - D), nv=nv + [1] * (3 - D), kappa=kappa, merge_kicks=merge)
    fa, la = _run(S, spec, storage, n, False)
    fb, lb = _run(S, spec, storage, n, True)
    assert lb == 0 and la == ((n + 1 if merge else 2 * n) if taken[storage] else 0)
    assert np.array_equal(fa, fb), np.abs(fa - fb).max()
    f0 = None
    if storage:
        f0 = O.init_separable(O.make_grid(spec), *W.separable_factors(spec)).astype(np.float32).astype(np.float64)
    run = O.Run(spec, f0)
    run.step(spec["dt"], n)
    err = np.abs(fa - run.f).sum() / max(np.abs(run.f).sum(), 1e-300)
    assert err <= (1e-12 if storage == 0 else 1e-5), err


@pytest.mark.parametrize("nx,nv,taken", [([46, 45], [31, 32], True), ([46, 46], [31, 32], False),
                                         ([46, 46], [32, 33], True)])
def test_rect_pass_on_large_grids(S, nx, nv, taken):
    """Either side of the size rule: 992-cell planes of a grid of 2.05e6 and
    of 2.10e6 cells (limit 2^21), 1056-cell planes of a larger one."""
    spec = W.landau_run(2, nx[0], nv[-1], 0.5, 0.3, 7)
    spec.update(nx=nx + [1], nv=nv + [1], kappa=-30.0)
    for storage in (0, 1):
        print(f"case rule nx={nx} nv={nv} storage={storage}", flush=True)
        fa, la = _run(S, spec, storage, 1, False)
        fb, lb = _run(S, spec, storage, 1, True)
        assert lb == 0 and la == (2 if taken else 0)
        assert np.array_equal(fa, fb)
