"""Velocity moments on both sides of the sizes from which a block is summed
through its marginals (directly below): blocks of two and three axes, planes of
31 and 32 cells, few large planes, 2047 and 2048 spatial cells.

Sums of at most N values of one sign in double, compensated above groups of
eight: 64 x 2^-53 relative for the density, that times the largest velocity for
the mean, four times that times its square for the dispersion."""
import numpy as np
import pytest

from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53
FEW = [[127, 129], [128, 128], [8, 8, 11], [8, 8, 12], [8, 16, 15], [8, 16, 16], [40, 31], [40, 32], [9, 1, 31],
       [7, 260], [8, 260]]
MANY = [[31, 66], [32, 64], [95, 97], [96, 96], [3, 256], [4, 256], [4, 31], [8, 8, 8]]
GRIDS = [(17, nv) for nv in FEW] + [(n, nv) for nv in MANY for n in (2047, 2048)] + [(5, [300]), (2050, [300])]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("gi", range(len(GRIDS)))
def test_moments(gi, storage):
    import torch

    from paper_1702_08521_amd import slmpp as S

    nxs, nv = GRIDS[gi]
    D = len(nv)
    print(f"case moments cells={nxs} nv={nv} storage={storage}", flush=True)
    spec = W.spec(D, [nxs] + [1] * (D - 1), nv, 0.0, 2.0, [-3.0 + l for l in range(D)], [4.0 + l for l in range(D)])
    ctx = S.Context(S.make_desc(spec, storage))
    gen = torch.Generator(device="cuda").manual_seed(gi)
    f = torch.rand(ctx.f.numel(), generator=gen, dtype=torch.float64, device="cuda").to(ctx.f.dtype)
    ctx.f.view(-1).copy_(f)
    new = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
    rho, mean, disp = new(nxs), new(D * nxs), new(D * nxs)
    ctx.velocity_moments(rho, mean, disp)
    ctx.close()
    g = f.cpu().numpy().astype(np.float64).reshape([nxs] + nv)
    hv = [(spec["v_hi"][l] - spec["v_lo"][l]) / nv[l] for l in range(D)]
    tot = g.reshape(nxs, -1).sum(1)
    assert (np.abs(rho.cpu().numpy() / np.prod(hv) - tot) <= 64 * EPS * tot).all()
    for l in range(D):
        v = spec["v_lo"][l] + (np.arange(nv[l]) + 0.5) * hv[l]
        m = g.sum(axis=tuple(1 + k for k in range(D) if k != l))
        u = (m * v).sum(1) / tot
        s2 = (m * (v - u[:, None]) ** 2).sum(1) / tot
        span = np.abs(v).max() + np.abs(u).max()
        assert np.abs(mean.cpu().numpy()[l * nxs:(l + 1) * nxs] - u).max() <= 64 * EPS * span
        assert np.abs(disp.cpu().numpy()[l * nxs:(l + 1) * nxs] - s2).max() <= 256 * EPS * span ** 2
