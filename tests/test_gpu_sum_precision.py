"""Sums over the velocity cells and over f hold a compensated pair above small
groups: two cells +-2^60 among ones must cancel without taking the ones along.

At most eight cells are added plainly before a compensated addition, so each of
the two cells costs at most the seven ones beside it; everything else is exact
(cells of unit volume): densities to 14, a mean velocity along an axis on which
the two cells agree to 14 times the largest velocity over the number of cells
for the numerator and as much for the denominator.  The diagnostics compensate
every value and are exact.  Row sums of an x sweep add vectors of at most four
cells plainly: the density to 6."""
import numpy as np
import pytest

from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu
BIG = 2.0 ** 60


@pytest.fixture(scope="module")
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_08521_amd import slmpp

    slmpp.lib()
    return slmpp


def _spec(nx, nv, **kw):
    return W.spec(len(nx), nx, nv, [0.0] * len(nx), [float(n) for n in nx], [0.0] * len(nv),
                  [float(n) for n in nv], **kw)


# blocks taken directly and through their marginals, by four wavefronts and by one
BLOCKS = [([3], [1000]), ([2, 2], [30, 41]), ([2, 2], [130, 131]), ([46, 45], [100, 100]), ([2, 2, 2], [8, 8, 8]),
          ([2, 2, 2], [24, 25, 26]), ([13, 13, 13], [12, 13, 14])]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("bi", range(len(BLOCKS)))
def test_velocity_moments(S, bi, storage):
    import torch

    nx, nv = BLOCKS[bi]
    D, nxs, nvs = len(nx), int(np.prod(nx)), int(np.prod(nv))
    ctx = S.Context(S.make_desc(_spec(nx, nv), storage))
    new = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
    rho, mean, disp = new(nxs), new(D * nxs), new(D * nxs)
    for axis in range(D):  # the axis on which the two cells agree
        print(f"case moments nx={nx} nv={nv} storage={storage} axis={axis}", flush=True)
        f = ctx.f.view(nxs, *nv)
        f.fill_(1.0)
        p, q = [n // 9 for n in nv], [n - 1 - n // 7 for n in nv]
        q[axis] = p[axis]
        if D == 1:
            q[0] = nv[0] - 2
        f[(slice(None), *p)] = BIG
        f[(slice(None), *q)] = -BIG
        ctx.velocity_moments(rho, mean, disp)
        n = nvs - 2
        assert np.abs(rho.cpu().numpy() - n).max() <= 14
        if D == 1:
            continue
        v = np.arange(nv[axis]) + 0.5
        ones = np.full(nv[axis], nvs / nv[axis])
        ones[p[axis]] -= 2
        ref = (ones * v).sum() / n
        got = mean.cpu().numpy()[axis * nxs:(axis + 1) * nxs]
        assert np.abs(got - ref).max() <= 2 * 14 * nv[axis] / (n - 14)
    ctx.close()


@pytest.mark.parametrize("storage", [0, 1])
def test_diagnostics(S, storage):
    ctx = S.Context(S.make_desc(_spec([7, 9], [30, 31]), storage))
    ctx.field()
    ctx.f.fill_(1.0)
    flat = ctx.f.view(-1)
    flat[10001] = BIG
    flat[41234] = -BIG
    print(f"case diagnostics storage={storage}", flush=True)
    assert ctx.diag()["mass"] == flat.numel() - 2
    ctx.close()


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("nx,nv", [([64], [128]), ([50], [611]), ([40, 50], [50, 53])])
def test_row_sums_of_the_x_sweep(S, nx, nv, storage):
    """A step of no duration keeps f; its density comes from the row sums."""
    import torch

    D = len(nx)
    ctx = S.Context(S.make_desc(_spec(nx, nv, kappa=0.0), storage))
    f = ctx.f.view(-1, int(np.prod(nv)))
    f.fill_(1.0)
    f[:, 11] = BIG
    f[:, 75] = -BIG
    before = ctx.f.clone()
    ctx.timing_enable(True)
    ctx.step(0.0, 1)
    assert ctx.timing_read()["sweep_x1_moment"]["launches"] == 1
    assert torch.equal(ctx.f, before)
    rho, _ = ctx.get_field()
    print(f"case row sums nx={nx} nv={nv} storage={storage}", flush=True)
    assert np.abs(rho - (np.prod(nv) - 2)).max() <= 6
    ctx.close()
