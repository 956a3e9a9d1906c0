"""The split backward projection with up to 64 columns (two waves along the columns): edges of its tiles and of k, d on
either side of its line, one plan.  Tolerance as for the wider ones: 22 bits of each operand and float32 sums of at most
256 terms, 1e-6 of the sum of an entry's terms' magnitudes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _error(dF, phi, mass, dA):
    scale = mass.astype(np.float64)[:, None] * (np.abs(phi).astype(np.float64) @ np.abs(dA).astype(np.float64))
    return float((np.abs(dF - np.asarray(oracle.project_backward(phi, mass, dA), np.float64)) / scale).max())


@pytest.mark.parametrize("b,n,k,d", [(3, 65, 4, 1), (2, 129, 5, 64), (2, 127, 31, 32), (1, 128, 32, 33), (2, 255, 33, 64),
                                     (1, 257, 64, 3), (2, 129, 65, 64), (1, 127, 95, 17), (2, 128, 97, 64), (1, 130, 127, 33),
                                     (2, 1, 128, 64), (2, 65, 193, 64), (1, 64, 223, 5), (2, 63, 225, 64), (1, 97, 256, 31),
                                     (40, 501, 70, 48), (2, 333, 160, 64), (2, 333, 300, 20), (2, 200, 100, 65)])
def test_tile_edges(dev, b, n, k, d):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(n + k)
    mass = rng.uniform(0.5, 1.5, (b, n)).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    dA = rng.standard_normal((b, k, d)).astype(np.float32)
    dF = F.fmap_project_backward(*(torch.from_numpy(x).to(dev) for x in (phi, mass, dA))).cpu().numpy()
    for s in {0, b - 1}:
        assert _error(dF[s], phi[s], mass[s], dA[s]) <= TOL


def test_plan(dev):
    """The items of a plan against the single calls (the solves may differ by their width: 1e-4)."""
    import torch
    from paper_2604_10377_amd import fmap as F
    g = torch.Generator(device=dev).manual_seed(3)
    rn = lambda *s: torch.randn(*s, generator=g, device=dev)
    pairs, d = [], 48
    for k, nx, ny in ((20, 700, 1301), (40, 650, 999), (20, 129, 64)):
        pairs.append(dict(phi_x=rn(nx, k), phi_y=rn(ny, k), mass_x=rn(nx).abs() / nx, mass_y=rn(ny).abs() / ny,
                          feat_x=rn(nx, d), feat_y=rn(ny, d), evals_x=torch.linspace(0, k, k, device=dev),
                          evals_y=torch.linspace(0, k, k, device=dev), lam=torch.full((1,), 0.1, device=dev)))
    plan = F.FmapPlan(pairs, want_AB=True)
    plan.forward()
    for dC in plan.dC:
        dC.copy_(rn(*dC.shape))
    plan.backward()
    torch.cuda.synchronize()
    for i, p in enumerate(pairs):
        A, B = plan.A[i][None], plan.B[i][None]
        _, fac, _, _ = F.fmap_solve(A, B, p["evals_x"][None], p["evals_y"][None], p["lam"])
        dA, dB, _ = F.fmap_solve_backward(plan.dC[i][None], A, B, plan.C[i][None], p["evals_x"][None], p["evals_y"][None],
                                          p["lam"], factors=fac)
        for x, grad, got in (("x", dA, plan.dF_x[i]), ("y", dB, plan.dF_y[i])):
            want = F.fmap_project_backward(p["phi_" + x][None], p["mass_" + x][None], grad)[0]
            assert (got - want).norm() <= 1e-4 * want.norm()
    plan.close()
