"""The velocity distribution on both sides of the numbers of spatial cells up
to which each velocity cell has one thread (above, vectors and shares).

Sums of values of one sign in double, compensated: 8 x 2^-53 relative."""
import numpy as np
import pytest

from paper_1702_08521_amd import workloads as W

pytestmark = pytest.mark.gpu
GRIDS = [(n, nv) for nv, ns in (([33], (1, 15, 16, 17)), ([31, 41], (127, 128, 129, 256, 257)),
                                ([96, 128], (511, 512, 513)), ([128, 257], (2047, 2048, 2049)))
         for n in ns]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("gi", range(len(GRIDS)))
def test_distribution(gi, storage):
    import torch

    from paper_1702_08521_amd import slmpp as S

    nxs, nv = GRIDS[gi]
    D, nvs = len(nv), int(np.prod(nv))
    print(f"case distribution cells={nxs} nv={nv} storage={storage}", flush=True)
    spec = W.spec(D, [nxs] + [1] * (D - 1), nv, 0.0, 2.0, -1.0, 1.0)
    ctx = S.Context(S.make_desc(spec, storage))
    gen = torch.Generator(device="cuda").manual_seed(gi)
    ctx.f.view(-1).copy_(torch.rand(ctx.f.numel(), generator=gen, dtype=torch.float64, device="cuda"))
    F = torch.full((nvs,), float("nan"), dtype=torch.float64, device="cuda")
    ctx.velocity_distribution(F)
    f = ctx.f.view(nxs, nvs).cpu().numpy().astype(np.longdouble)
    ctx.close()
    ref = f.sum(0) * np.longdouble(2.0 / nxs) * 2.0 ** (D - 1)
    assert (np.abs(F.cpu().numpy() - ref) <= 8 * 2.0 ** -53 * ref).all()
