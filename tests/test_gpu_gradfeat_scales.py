"""Gradient features on the split matrix-core kernel: tile edges, and rows and weights far apart in scale.

Tolerance per vertex: both operands keep 22 bits and the sums (at most 512 terms) are float32, so the transformed
parts are within 1e-6 of their largest terms; g sums two products of them, whose cancellation the bound covers by
measuring against sum_j |A_cj| |z_j| |z_c| instead of |g|.
"""
import numpy as np
import pytest

from oracle import gradfeat as gf

pytestmark = pytest.mark.gpu
TOL = 1e-6


@pytest.mark.parametrize("variant", ["A", "B"])
@pytest.mark.parametrize("V,D", [(127, 32), (129, 32), (63, 64), (65, 64), (31, 128), (33, 128), (8300, 128), (32, 256),
                                 (49, 256)])
def test_rows_and_weights_of_any_scale(dev, V, D, variant):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(V + D)
    z = rng.standard_normal((V, D, 2)) * np.logspace(-12, 12, V)[:, None, None]
    z[V // 2] = 0
    Ar = rng.standard_normal((D, D)) * np.logspace(-6, 6, D)[:, None]
    Ai = rng.standard_normal((D, D)) * np.logspace(-6, 6, D)[:, None]
    Ar[1], Ai[1] = 0, 0
    z, Ar, Ai = (np.ascontiguousarray(a, np.float32) for a in (z, Ar, Ai))
    g = F.fmap_gradient_features(*(torch.from_numpy(a).to(dev) for a in (z, Ar, Ai)), variant).cpu().numpy()
    ref = gf.gradient_features(z, Ar, Ai, variant)
    mag = np.abs(z.astype(np.float64)).sum(2)
    scale = mag * (mag @ (np.abs(Ar) + np.abs(Ai)).astype(np.float64).T)
    assert np.all(np.abs(g - ref) <= TOL * scale)
