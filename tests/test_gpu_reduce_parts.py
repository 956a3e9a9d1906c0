"""The sum over a short forward projection's chunks (k <= 64), where four waves share it and on either side of that rule:
64, 65 and more chunks, fewer elements than a wave, the last element count that one workgroup per CU covers and the next.

Tolerance, per entry: float32 sums of at most 32 stages and 156 chunks, a few 2^-24 sqrt(chunks) of the sum of the entry's
terms' magnitudes, and operands of 22 bits: 2e-6.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n,k,d", [(1, 8256, 5, 12), (1, 8320, 5, 12), (1, 8321, 1, 4), (3, 9301, 3, 28),
                                     (2, 20000, 30, 256), (1, 20000, 1, 4), (1, 19999, 33, 300), (2, 8400, 64, 512),
                                     (2, 8400, 64, 516), (4, 49998, 4, 16)])
def test_sum_over_chunks(dev, b, n, k, d):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(n + k)
    mass = (rng.uniform(0.5, 1.5, (b, n)) / n).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    feat = rng.standard_normal((b, n, d)).astype(np.float32)
    t = [torch.from_numpy(x).to(dev) for x in (phi, mass, feat)]
    A = F.fmap_project(*t)
    assert torch.equal(A, F.fmap_project(*t))
    A = A.cpu().numpy()
    for s in range(b):
        scale = (np.abs(phi[s]) * mass[s][:, None]).T.astype(np.float64) @ np.abs(feat[s])
        assert (np.abs(A[s] - np.asarray(oracle.project(phi[s], mass[s], feat[s]))) / scale).max() <= 2e-6
