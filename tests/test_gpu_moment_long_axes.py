"""Velocity moments whose marginals do not fit the LDS and, over all spatial
cells, not the scratch either: the cells are taken in several launches.

f = s(x) g1(v1) g3(v3) rounded once to FP32 (2^-24 relative): the density is
right to 2^-24 of itself, a mean velocity to twice that times the largest
velocity, a dispersion to four times that times the largest velocity squared
(numerator, denominator and mean)."""
import numpy as np
import pytest

from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_marginals_of_more_cells_than_the_scratch_holds():
    import torch

    from paper_1702_08521_amd import slmpp as S

    nx, nv = [280, 1, 1], [4096, 1, 3413]
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GiB of device memory")
    print(f"case moments nx={nx} nv={nv}", flush=True)
    spec = W.spec(3, nx, nv, 0.0, 1.0, [-3.0, -1.0, -2.0], [5.0, 1.0, 2.5])
    rng = np.random.default_rng(1)
    sx = 1.0 + rng.random(280)
    h = [(spec["v_hi"][l] - spec["v_lo"][l]) / nv[l] for l in range(3)]
    v = [spec["v_lo"][l] + (np.arange(nv[l]) + 0.5) * h[l] for l in range(3)]
    g = [np.exp(-0.5 * (v[l] - 0.3) ** 2) * (1.0 + 0.1 * rng.random(nv[l])) for l in range(3)]
    ctx = S.Context(S.make_desc(spec, S.F32))
    ctx.init_f_separable(sx, g)
    new = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
    rho, mean, disp = new(280), new(3 * 280), new(3 * 280)
    ctx.velocity_moments(rho, mean, disp)
    ref = sx * g[0].sum() * g[1].sum() * g[2].sum() * np.prod(h)
    e = 2.0 ** -24
    assert (np.abs(rho.cpu().numpy() - ref) <= e * ref).all()
    for l in range(3):
        u = (g[l] * v[l]).sum() / g[l].sum()
        d = (g[l] * (v[l] - u) ** 2).sum() / g[l].sum()
        big = np.abs(v[l]).max()
        assert np.abs(mean.cpu().numpy()[l * 280:(l + 1) * 280] - u).max() <= 2 * e * big
        assert np.abs(disp.cpu().numpy()[l * 280:(l + 1) * 280] - d).max() <= 4 * e * (2 * big) ** 2
    ctx.close()
