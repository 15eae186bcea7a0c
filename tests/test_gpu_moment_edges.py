"""Velocity moments, velocity distribution and diagnostics at the edges of
their kernels' shapes: velocity planes shorter than a 16-byte vector, planes
that end within a vector, one plane per wavefront pass and several, several
chunks per plane with a remainder, few spatial cells (four wavefronts each)
and many (one each), the spatial cells dealt to several shares, and
non-finite values within a vector and in the last cells.

Bounds: every sum is compensated or runs over a few dozen values, so the
results agree with numpy's 64-bit pairwise sums to 64 roundings (64 * 2^-53
relative to the sum of magnitudes) before the two divisions; the dispersion
is a sum of squares with no cancellation against its own size beyond the
spread of the axis, hence the same bound times the square of the axis
length over the dispersion."""
import numpy as np
import pytest

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


GRIDS = [
    (1, [5], [1]), (1, [3], [3]), (1, [7], [259]), (1, [2500], [34]),
    (2, [3, 2], [5, 1]), (2, [3, 5], [9, 3]), (2, [6, 6], [7, 130]), (2, [64, 33], [10, 17]),
    (3, [2, 3, 2], [4, 1, 2]), (3, [3, 2, 4], [9, 23, 25]), (3, [2, 2, 2], [33, 40, 40]),
    (3, [13, 13, 13], [5, 6, 7]), (3, [13, 13, 13], [3, 24, 24]),
]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("gi", range(len(GRIDS)))
def test_moments_distribution_diag(S, gi, storage):
    import torch

    D, nx, nv = GRIDS[gi]
    spec = W.spec(D, nx, nv, 0.0, 2.0, [-3.0 + l for l in range(D)], [4.0 + l for l in range(D)])
    shape = tuple(nx) + tuple(nv)
    f = W.random_field(shape, 100 + gi, zeros=0.1, spikes=0.02)
    f = f.astype(np.float32).astype(np.float64) if storage else f
    print(f"case D={D} nx={nx} nv={nv} storage={storage}", flush=True)
    ctx = S.Context(S.make_desc(spec, storage))
    ctx.init_f_host(f)
    nxs, nvs = int(np.prod(nx)), int(np.prod(nv))
    new = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
    rho, mean, disp, F = new(nxs), new(D * nxs), new(D * nxs), new(nvs)
    ctx.velocity_moments(rho, mean, disp)
    ctx.velocity_distribution(F)
    d = ctx.diag()
    g = f.reshape([nxs] + nv)
    hv = [(spec["v_hi"][l] - spec["v_lo"][l]) / nv[l] for l in range(D)]
    tot = g.reshape(nxs, -1).sum(1)
    assert np.abs(rho.cpu().numpy() - tot * np.prod(hv)).max() <= 64 * EPS * tot.max() * np.prod(hv)
    for l in range(D):
        v = spec["v_lo"][l] + (np.arange(nv[l]) + 0.5) * hv[l]
        m = g.sum(axis=tuple(1 + k for k in range(D) if k != l))
        live = tot > 0
        u = np.where(live, (m * v).sum(1) / np.where(live, tot, 1.0), 0.0)
        s2 = np.where(live, (m * (v - u[:, None]) ** 2).sum(1) / np.where(live, tot, 1.0), 0.0)
        span = np.abs(v).max() + np.abs(u).max()
        assert np.abs(mean.cpu().numpy()[l * nxs:(l + 1) * nxs] - u).max() <= 64 * EPS * span
        assert np.abs(disp.cpu().numpy()[l * nxs:(l + 1) * nxs] - s2).max() <= 256 * EPS * span ** 2
    ref = f.reshape(nxs, -1).sum(0) * (2.0 / np.array(nx)).prod()
    assert np.abs(F.cpu().numpy() - ref).max() <= 64 * EPS * ref.max()
    vol = np.prod(hv) * (2.0 / np.array(nx)).prod()
    assert abs(d["mass"] - f.sum() * vol) <= 64 * EPS * f.sum() * vol
    assert d["f_min"] == f.min() and d["f_max"] == f.max() and d["nonfinite"] == 0
    # a few non-finite values: counted, and nothing else changes by them
    flat = ctx.f.view(-1)
    at = sorted({0, flat.numel() // 2, flat.numel() - 1})
    flat[at[0]] = float("nan")
    for k, q in enumerate(at[1:]):
        flat[q] = float("-inf") if k else float("inf")
    ctx.field()
    d = ctx.diag()
    rest = np.delete(f.ravel(), at)
    assert d["nonfinite"] == len(at)
    if rest.size:
        assert d["f_min"] == rest.min() and d["f_max"] == rest.max()
    assert abs(d["mass"] - rest.sum() * vol) <= 64 * EPS * f.sum() * vol
    ctx.close()
