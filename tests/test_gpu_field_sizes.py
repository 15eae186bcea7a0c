"""The field solve where its path changes: one-dimensional axes over 1024 cells
and up to the longest (odd, even, prime), and grids with one long axis beside
short ones, periodic and isolated, which are solved in a launch per axis rather
than in four launches; outputs on top of the density there as well.

Against the FP64 oracle: 32 n roundings of the largest potential (the angles of
the roots of unity near 2 pi carry n roundings), and what that makes of a
force, a difference of potentials over 60 h / 110."""
import numpy as np
import pytest

import oracle as O
from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53
SOLVES = [([1025], 6, 0), ([1100], 4, 0), ([2047], 6, 0), ([2048], 2, 0), ([4096], 6, 0), ([4, 601], 6, 0),
          ([3, 20, 50], 6, 0), ([4, 45, 45], 4, 0), ([8, 8, 32], 6, 1), ([6, 6, 48], 4, 1), ([40, 6, 6], 6, 1)]


@pytest.mark.parametrize("i", range(len(SOLVES)))
def test_solve(i):
    import torch

    from paper_1702_08521_amd import slmpp as S

    nx, order, isolated = SOLVES[i]
    D, nxs = len(nx), int(np.prod(nx))
    hi = [1.0 + 0.3 * l for l in range(D)]
    spec = W.spec(D, nx, [2] * D, [0.0] * D, hi, -1.0, 1.0, kappa=4 * np.pi if isolated else -1.0,
                  poisson_order=order, field_bc="isolated" if isolated else "periodic")
    grid = O.make_grid(spec)
    rho = 1.0 + np.random.default_rng(nxs + order).random(nxs)
    po, ao = O.poisson_isolated(grid, rho) if isolated else O.poisson_solve(grid, rho)
    tol = 32 * max(nx) * EPS * np.abs(po).max()
    ctx = S.Context(S.make_desc(spec, 0))
    for in_place in (False, True):
        print(f"case solve nx={nx} order={order} isolated={isolated} in_place={in_place}", flush=True)
        r = torch.tensor(rho, dtype=torch.float64, device="cuda")
        acc = torch.full((D * nxs,), float("nan"), dtype=torch.float64, device="cuda")
        phi = r if in_place else torch.full((nxs,), float("nan"), dtype=torch.float64, device="cuda")
        ctx.poisson_solve(r, acc, phi)
        ctx.sync()
        assert np.abs(phi.cpu().numpy() - po).max() <= tol
        for l in range(D):
            err = np.abs(acc.cpu().numpy()[l * nxs:(l + 1) * nxs] - ao[l * nxs:(l + 1) * nxs]).max()
            assert err <= 2 * tol * 110.0 / (60.0 * hi[l] / nx[l])
    ctx.close()
