"""The forward projection for k > 64 on either side of the line between small calls (the sliced kernel) and larger ones
(the tall kernel), which lies at 2.5, 5 and 4 stages of 32 vertices per CU and column block, and small calls with odd
last stages.

Tolerance, per entry: float32 sums of at most 32 stages, a few 2^-24 sqrt(stages) of the sum of the entry's terms'
magnitudes, and operands of 22 bits or more: 2e-6.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n,k,d", [(20, 992, 72, 100), (20, 1024, 72, 100), (20, 992, 100, 260), (20, 1024, 100, 260),
                                     (16, 992, 200, 256), (16, 1024, 200, 256), (1, 128, 68, 88), (3, 500, 128, 512),
                                     (2, 1004, 256, 320), (1, 132, 316, 396)])
def test_both_sides(dev, b, n, k, d):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(n + k)
    mass = (rng.uniform(0.5, 1.5, (b, n)) / n).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    feat = rng.standard_normal((b, n, d)).astype(np.float32)
    A = F.fmap_project(*(torch.from_numpy(x).to(dev) for x in (phi, mass, feat))).cpu().numpy()
    for s in {0, b - 1}:
        scale = (np.abs(phi[s]) * mass[s][:, None]).T.astype(np.float64) @ np.abs(feat[s])
        assert (np.abs(A[s] - np.asarray(oracle.project(phi[s], mass[s], feat[s]))) / scale).max() <= 2e-6
