"""Maps at several resolutions whose normal products come from one covering resolution are the maps of the
single-resolution calls, bit for bit (the same sums entry by entry): the covering one in place or smaller than the
inputs, more resolutions than one gather launch takes, repeats, rectangular ones, and lists that nothing covers."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [0, 1])
@pytest.mark.parametrize("P,kx,ky,d,res", [
    (3, 120, 120, 256, [(30, 30), (50, 50), (80, 80), (120, 120)]),
    (2, 130, 100, 200, [(65, 64), (129, 97), (33, 97), (129, 2), (64, 64)]),
    (2, 40, 70, 90, [(40, 70), (40, 70), (2, 3)] + [(40 - i, 70 - 2 * i) for i in range(1, 12)]),
    (2, 70, 70, 99, [(70, 20), (20, 70), (35, 35)]),
    (1, 2, 1, 5, [(2, 1), (1, 1)]),
])
def test_resolutions_from_shared_products(dev, mask, P, kx, ky, d, res):
    import torch
    from paper_2604_10377_amd import fmap as F
    g = torch.Generator(device=dev).manual_seed(5)
    A, B = torch.randn(P, kx, d, generator=g, device=dev), torch.randn(P, ky, d, generator=g, device=dev)
    ex, ey = ((torch.rand(P, k, generator=g, device=dev) * 50 + 0.1).sort(1).values for k in (kx, ky))
    lam = torch.rand(P, generator=g, device=dev) + 0.01
    print("resolutions", P, kx, ky, d, res[:4], flush=True)
    out = F.fmap_solve_resolutions(A, B, ex, ey, lam, mask, 0.5, res)
    for (C, info), r in zip(out, res):
        (C1, info1), = F.fmap_solve_resolutions(A, B, ex, ey, lam, mask, 0.5, [r])
        assert (info == 0).all() and torch.equal(info, info1), r
        assert torch.isfinite(C).all() and torch.equal(C, C1), r
