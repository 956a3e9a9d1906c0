"""The split forward projection for k <= 64 (float32, any n and k): edges of its windows, stages and scales.

Tolerance: the two-part float16 products keep 22 bits of each operand and sums are float32, so an entry is within a
few 2^-24 sqrt(terms) of the float64 one, relative to the sum of its terms' magnitudes (an entry whose terms cancel is
no more exact than they are): 2e-6 leaves room for 40 stages.  A chunk computed again by the general float32 routine
sums one vertex pair at a time: 4e-6.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 2e-6


def _run(dev, *arrays):
    import torch
    from paper_2604_10377_amd import fmap as F
    return F.fmap_project(*(torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(dev) for x in arrays)).cpu().numpy()


def _error(A, phi, mass, feat):
    """Largest error of an entry, relative to the sum of its terms' magnitudes."""
    scale = (np.abs(phi).astype(np.float64) * mass[:, None]).T @ np.abs(feat).astype(np.float64)
    err = np.abs(A - np.asarray(oracle.project(phi, mass, feat), np.float64))
    assert np.all(err[scale == 0] == 0)
    return float((err / np.where(scale > 0, scale, 1)).max())


@pytest.mark.parametrize("b,n,k,d", [(3, 128, 1, 4), (2, 131, 3, 8), (2, 999, 17, 36), (1, 1001, 31, 260), (2, 645, 32, 128),
                                     (3, 1503, 33, 64), (2, 4999, 49, 256), (2, 803, 50, 512), (1, 1307, 57, 388),
                                     (2, 2049, 63, 128), (1, 1310, 64, 252)])
def test_window_edges(dev, b, n, k, d):
    rng = np.random.default_rng(100 + k)
    mass = rng.uniform(0.5, 1.5, (b, n)).astype(np.float32) / np.float32(n)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    feat = rng.standard_normal((b, n, d)).astype(np.float32)
    A = _run(dev, phi, mass, feat)
    for s in range(b):
        assert _error(A[s], phi[s], mass[s], feat[s]) <= TOL


@pytest.mark.parametrize("kind", ["growing", "sparse", "column scales", "late column", "infinite"])
def test_scales_and_the_general_routine(dev, kind):
    """Columns far apart in scale stay on the split path; values that outgrow it take the general routine."""
    n, k, d = 1700, 45, 300
    rng = np.random.default_rng(12)
    mass = (rng.uniform(0.5, 1.5, n) / n).astype(np.float32)
    phi = rng.standard_normal((n, k))
    feat = rng.standard_normal((n, d))
    if kind == "growing":
        feat *= np.logspace(-9, 9, n)[:, None]
    elif kind == "sparse":
        feat *= rng.uniform(size=(n, d)) < 0.02
    elif kind == "column scales":
        feat *= np.logspace(-25, 25, d)[None, :]
        phi *= np.logspace(-6, 6, k)[None, :]
    elif kind == "late column":
        feat[:1000, 7] = 0
        feat[1000:, 7] *= 1e20
    phi, feat = phi.astype(np.float32), feat.astype(np.float32)
    if kind == "infinite":
        feat[900, 11] = np.inf
    A = _run(dev, phi[None], mass[None], feat[None])[0]
    if kind == "infinite":
        assert np.array_equal(np.sign(A[:, 11]), np.sign(phi[900])) and np.isinf(A[:, 11]).all()
        A, feat = np.delete(A, 11, 1), np.delete(feat, 11, 1)
    assert _error(A, phi, mass, feat) <= 2 * TOL
