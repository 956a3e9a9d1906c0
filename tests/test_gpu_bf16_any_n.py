"""The bf16 forward projection at vertex counts that are no multiple of 4 (three bf16 parts of basis x mass): every
remainder, row-slab width and a last stage of one vertex; shapes that start at any 4-byte mass address.

Tolerance: three parts keep 24 bits of basis x mass, the bf16 features are exact and sums are float32, so an entry is
within a few 2^-24 sqrt(stages) of the float64 one, relative to the sum of its terms' magnitudes: 2e-6."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 2e-6


@pytest.mark.parametrize("b,n,k,d", [(3, 129, 8, 8), (2, 1001, 64, 520), (3, 1602, 96, 136), (2, 2047, 128, 256),
                                     (3, 1283, 200, 384), (2, 5009, 256, 72), (1, 30001, 160, 128)])
def test_any_vertex_count(dev, b, n, k, d):
    import torch
    from paper_2604_10377_amd import fmap as F
    g = torch.Generator().manual_seed(n)
    phi, feat = (torch.randn(b, n, c, generator=g).bfloat16() for c in (k, d))
    mass = (0.5 + torch.rand(b, n, generator=g)) / n
    print("bf16 projection", b, n, k, d, flush=True)
    A = F.fmap_project(phi.to(dev), mass.to(dev), feat.to(dev)).cpu().numpy()
    for s in range(b):
        x, m, f = phi[s].double().numpy(), mass[s].double().numpy(), feat[s].double().numpy()
        scale = (np.abs(x) * m[:, None]).T @ np.abs(f)
        assert (np.abs(A[s] - oracle.project(x, m, f)) / scale).max() <= TOL
