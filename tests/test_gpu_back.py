"""The split backward projection (float32, 4 <= k <= 319, any n, k and d): edges of its tiles, chunks of k and scales.

Tolerance: both operands keep 22 bits and the sums (at most 319 terms) are float32, so an entry is within a few 2^-24
of the sum of its terms' magnitudes: 1e-6.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _run(dev, *arrays):
    import torch
    from paper_2604_10377_amd import fmap as F
    return F.fmap_project_backward(*(torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(dev) for x in arrays)).cpu().numpy()


def _error(dF, phi, mass, dA):
    scale = mass.astype(np.float64)[:, None] * (np.abs(phi).astype(np.float64) @ np.abs(dA).astype(np.float64))
    err = np.abs(dF - np.asarray(oracle.project_backward(phi, mass, dA), np.float64))
    assert np.all(err[scale == 0] == 0)
    return float((err / np.where(scale > 0, scale, 1)).max())


@pytest.mark.parametrize("b,n,k,d", [(2, 1, 4, 1), (3, 65, 5, 3), (2, 31, 32, 33), (1, 129, 33, 130), (2, 999, 49, 256),
                                     (3, 257, 63, 128), (1, 100, 64, 257), (2, 333, 65, 96), (1, 96, 97, 384),
                                     (2, 511, 127, 256), (1, 301, 129, 100), (2, 222, 191, 256), (1, 77, 193, 64),
                                     (2, 401, 199, 256), (1, 130, 226, 300), (2, 65, 257, 512), (1, 500, 319, 132)])
def test_tile_edges(dev, b, n, k, d):
    rng = np.random.default_rng(200 + k)
    mass = rng.uniform(0.5, 1.5, (b, n)).astype(np.float32)
    phi = rng.standard_normal((b, n, k)).astype(np.float32)
    dA = rng.standard_normal((b, k, d)).astype(np.float32)
    dF = _run(dev, phi, mass, dA)
    for s in range(b):
        assert _error(dF[s], phi[s], mass[s], dA[s]) <= TOL


@pytest.mark.parametrize("k", [30, 299])
def test_rows_and_columns_of_any_scale(dev, k):
    n, d = 211, 140
    rng = np.random.default_rng(k)
    mass = (rng.uniform(0.5, 1.5, n) * np.logspace(-5, 0, n)).astype(np.float32)
    phi = (rng.standard_normal((n, k)) * np.logspace(-10, 10, n)[:, None]).astype(np.float32)
    dA = (rng.standard_normal((k, d)) * np.logspace(-15, 15, d)[None, :]).astype(np.float32)
    phi[17] = 0
    dA[:, 19] = 0
    assert _error(_run(dev, phi[None], mass[None], dA[None])[0], phi, mass, dA) <= TOL
