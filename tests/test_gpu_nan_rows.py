"""A NaN in the basis reaches its own row of the forward projection and no other: the last values of the last vertex,
which the kernels repeat to fill the last stage of 32 vertices.

Tolerance of the other entries, relative to the sum of their terms' magnitudes: 2e-6 as in the kernels' own tests, and
2^-16 of the two-part bf16 kernel's basis x mass (vertex counts that are multiples of 4).
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,d,bf16", [(221, 45, 128, False), (220, 64, 256, False), (129, 7, 36, False),
                                        (221, 120, 256, False), (220, 120, 128, False), (223, 48, 64, True),
                                        (221, 120, 256, True), (220, 200, 128, True), (129, 8, 8, True)])
def test_nan_stays_in_its_row(dev, n, k, d, bf16):
    import torch
    from paper_2604_10377_amd import fmap as F
    g = torch.Generator().manual_seed(n + k)
    phi, feat = torch.randn(n, k, generator=g), torch.randn(n, d, generator=g)
    mass = (0.5 + torch.rand(n, generator=g)) / n
    phi[n - 1, k - 1] = float("nan")
    if bf16:
        phi, feat = phi.bfloat16(), feat.bfloat16()
    A = F.fmap_project(phi.to(dev)[None], mass.to(dev)[None], feat.to(dev)[None])[0].cpu().numpy()
    assert np.isnan(A[k - 1]).all()
    x, m, f = phi.double().numpy()[:, :k - 1], mass.double().numpy(), feat.double().numpy()
    scale = (np.abs(x) * m[:, None]).T @ np.abs(f)
    assert (np.abs(A[:k - 1] - oracle.project(x, m, f)) / scale).max() <= (2.0 ** -16 if bf16 and n % 4 == 0 else 2e-6)
