"""slmpp_poisson_solve with an output on top of the density: the whole density
is read before any of it is overwritten, so the results are those of separate
arrays bit for bit, on every path of the solve (the one-dimensional
convolution from one workgroup to many, the transforms beyond it, two and
three dimensions, isolated boundaries)."""
import numpy as np
import pytest

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


GRIDS = [([16], 0), ([17], 0), ([255], 0), ([1024], 0), ([1030], 0), ([30, 37], 0), ([6, 5, 7], 0), ([9, 8, 6], 1)]


@pytest.mark.parametrize("nx,isolated", GRIDS)
def test_outputs_on_top_of_the_density(S, nx, isolated):
    import torch

    D, nxs = len(nx), int(np.prod(nx))
    spec = W.spec(D, nx, [2] * D, 0.0, 1.3, -1.0, 1.0,
                  field_bc="isolated" if isolated else "periodic")
    ctx = S.Context(S.make_desc(spec, 0))
    rho = torch.tensor(1.0 + np.random.default_rng(nxs).random(nxs), device="cuda")
    new = lambda n: torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
    phi, acc = new(nxs), new(D * nxs)
    ctx.poisson_solve(rho, acc, phi)
    print(f"case in place nx={nx} isolated={isolated}", flush=True)
    # phi on the density
    r, a = rho.clone(), new(D * nxs)
    ctx.poisson_solve(r, a, r)
    assert torch.equal(r, phi) and torch.equal(a, acc)
    # the first acceleration component on the density, with and without phi
    for with_phi in (True, False):
        buf, p = new(D * nxs), new(nxs)
        buf[:nxs] = rho
        ctx.poisson_solve(buf, buf, p if with_phi else None)
        assert torch.equal(buf, acc) and (not with_phi or torch.equal(p, phi))
    # partly on the density: half of it, from below and from above
    h = nxs // 2
    buf, a = new(nxs + h), new(D * nxs)
    buf[h:] = rho
    ctx.poisson_solve(buf[h:], a, buf[:nxs])
    assert torch.equal(buf[:nxs], phi) and torch.equal(a, acc)
    buf, p = new(h + D * nxs), new(nxs)
    buf[:nxs] = rho
    ctx.poisson_solve(buf[:nxs], buf[h:], p)
    assert torch.equal(buf[h:], acc) and torch.equal(p, phi)
    ctx.close()
