"""The tall forward projection (float32, 64 < k <= 319, any n and k): edges of its tiles, chunks and scales.

Tolerance: the two-part float16 products keep 22 bits of each operand and sums are float32, so each chunk's sums
are within a few 2^-24 sqrt(terms) of the float64 ones, column by column: 2e-6 leaves room for 40 stages.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 2e-6


def _columns_error(A, ref):
    ref = np.asarray(ref, np.float64)
    return float((np.linalg.norm(A - ref, axis=0) / np.linalg.norm(ref, axis=0)).max())


@pytest.mark.parametrize("b,n,k,d", [(2, 128, 65, 4), (1, 161, 128, 260), (3, 999, 129, 36), (1, 1501, 192, 128),
                                     (2, 640, 193, 132), (1, 2177, 256, 64), (2, 803, 257, 512), (1, 1301, 319, 388)])
def test_tile_edges(dev, b, n, k, d):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(k)
    mass = (rng.uniform(0.5, 1.5, (b, n)) / n).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    feat = rng.standard_normal((b, n, d)).astype(np.float32)
    A = F.fmap_project(*(torch.from_numpy(x).to(dev) for x in (phi, mass, feat))).cpu().numpy()
    for s in range(b):
        assert _columns_error(A[s], oracle.project(phi[s], mass[s], feat[s])) <= TOL


@pytest.mark.parametrize("kind", ["growing", "sparse", "column scales", "zero column"])
def test_scales_follow_the_values(dev, kind):
    """Values that outgrow the scale of the first stage, columns far apart in scale, columns of zeros."""
    import torch
    from paper_2604_10377_amd import fmap as F
    n, k, d = 1700, 70, 64
    rng = np.random.default_rng(11)
    mass = (rng.uniform(0.5, 1.5, n) / n).astype(np.float32)
    phi = rng.standard_normal((n, k))
    feat = rng.standard_normal((n, d))
    if kind == "growing":
        feat *= np.logspace(-9, 9, n)[:, None]
        phi *= np.logspace(-6, 6, k)[None, :]
    elif kind == "sparse":
        feat *= rng.uniform(size=(n, d)) < 0.02
    elif kind == "column scales":
        feat *= np.logspace(-25, 25, d)[None, :]
    else:
        feat[:, 5] = 0
    phi, feat = phi.astype(np.float32), feat.astype(np.float32)
    A = F.fmap_project(*(torch.from_numpy(x[None]).to(dev) for x in (phi, mass, feat)))[0].cpu().numpy()
    ref = oracle.project(phi, mass, feat)
    if kind == "zero column":
        assert not A[:, 5].any()
        A, ref = np.delete(A, 5, 1), np.delete(ref, 5, 1)
    if kind == "growing":  # rows far apart too: every row and column by itself
        assert _columns_error(A.T, np.asarray(ref).T) <= TOL
    assert _columns_error(A, ref) <= TOL
