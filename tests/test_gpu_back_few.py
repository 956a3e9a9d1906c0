"""The backward projection for k = 1, 2, 3 (a stream of dF): columns that fill a workgroup, leave lanes idle or need several,
rows at the edges of a workgroup's run, rows that are not 16-byte aligned.

Tolerance, per entry: four float32 roundings of at most three products, 4 * 2^-24 of the sum of their magnitudes: 3e-7.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("b,n,d,off", [(1, 1, 1, 0), (3, 85, 3, 0), (2, 1025, 3, 0), (2, 65, 16, 0), (2, 129, 100, 0),
                                       (2, 203, 200, 0), (1, 64, 255, 0), (2, 33, 257, 0), (1, 31, 1024, 0), (2, 17, 1028, 0),
                                       (2, 129, 64, 1), (90, 1500, 36, 0)])
def test_few_columns_of_the_basis(dev, k, b, n, d, off):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(n + k)
    mass = rng.uniform(0.5, 1.5, (b, n)).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    dA = rng.standard_normal((b, k, d)).astype(np.float32)
    g = torch.empty(b * k * d + off, device=dev)[off:].view(b, k, d).copy_(torch.from_numpy(dA))
    dF = F.fmap_project_backward(torch.from_numpy(phi).to(dev), torch.from_numpy(mass).to(dev), g).cpu().numpy()
    for s in range(0, b, 30):
        scale = mass[s].astype(np.float64)[:, None] * (np.abs(phi[s]).astype(np.float64) @ np.abs(dA[s]))
        want = np.asarray(oracle.project_backward(phi[s], mass[s], dA[s]), np.float64)
        assert (np.abs(dF[s] - want) / scale).max() <= 3e-7
    assert np.isfinite(dF).all()
