"""The tile shapes of the square-plane kick pass: planes in fours, twos and
ones, by the number of planes that share a spatial cell (1, 2, 3, 4, 6), with
tiles that end within a cell, a last tile that is not full, mirrored sweeps and
shifts beyond the ring of zero cells.  The pass and SLMPP_FLAG_SEPARATE_KICKS
perform the same operations on every pencil: identical bit for bit."""
import numpy as np
import pytest

from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("n", [24, 32])
@pytest.mark.parametrize("vouter", [1, 2, 3, 4, 6])
def test_plane_shapes(vouter, n, order, storage):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08521_amd import slmpp as S

    D = 2 if vouter == 1 else 3
    nx = [3, 3, 3][:D]  # an odd number of planes unless vouter is even
    spec = W.landau_run(D, 4, n, 0.5, 0.3, order)
    spec.update(nx=nx + [1] * (3 - D), nv=([vouter, n, n] if D == 3 else [n, n]) + [1] * (3 - D))
    f0 = W.random_field(nx + spec["nv"][:D], 7 * n + vouter)
    dt = 0.1
    # shifts of both signs, within the ring of 4 cells and up to 15 cells
    out = []
    for kappa in (-0.03, -0.3):
        for separate in (False, True):
            print(f"case vouter={vouter} n={n} order={order} storage={storage} kappa={kappa}", flush=True)
            s = dict(spec, separate_kicks=separate, kappa=kappa)
            ctx = S.Context(S.make_desc(s, storage))
            ctx.init_f_host(f0)
            ctx.timing_enable(True)
            ctx.step(dt, 2)
            assert ctx.timing_read()["kick_plane"]["launches"] == (0 if separate else 4)
            out.append(ctx.get_f())
            ctx.close()
        assert np.isfinite(out[-1]).all() and np.array_equal(out[-2], out[-1])
    assert not np.array_equal(out[0], out[2])
