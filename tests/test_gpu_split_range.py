"""Values far apart along the index that is summed over, on the two-part float16 products: what include/fmap.h states.

An operand value keeps 22 bits where it is within 2^-11 (forward) or 2^-17 (backward, gradient features) of the largest
one that shares its scale, and is otherwise off by at most 2^-34 (2^-38) of that one.  So an entry is within a few 2^-24
of the sum of its terms' magnitudes (the kernels' own tests: 2e-6, 1e-6) plus that floor times the sum of the other
operand's magnitudes, twice over for the two operands' roundings.
"""
import numpy as np
import pytest

import oracle
from oracle import gradfeat as gf

pytestmark = pytest.mark.gpu


def _spread(rng, count, decades):
    return 10.0 ** rng.uniform(-decades / 2, decades / 2, count)


def _floor(a, b, bits):
    """2^-bits (max|a| sum|b| + sum|a| max|b|) for a [rows][terms] and b [terms][columns]."""
    a, b = np.abs(a).astype(np.float64), np.abs(b).astype(np.float64)
    return 2.0 ** -bits * (a.max(1)[:, None] * b.sum(0)[None, :] + a.sum(1)[:, None] * b.max(0)[None, :])


@pytest.mark.parametrize("decades", [2, 8, 16])
@pytest.mark.parametrize("n,k,d", [(700, 45, 128), (701, 120, 256), (3001, 300, 384)])
def test_forward(dev, n, k, d, decades):
    """Vertices apart: basis rows times s_v, feature rows divided by s_v."""
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(decades + k)
    s = _spread(rng, n, decades)[:, None]
    phi = (rng.standard_normal((n, k)) * s).astype(np.float32)
    feat = (rng.standard_normal((n, d)) / s).astype(np.float32)
    mass = np.full(n, 1.0 / 1024, np.float32)
    A = F.fmap_project(*(torch.from_numpy(x[None]).to(dev) for x in (phi, mass, feat)))[0].cpu().numpy()
    err = np.abs(A - np.asarray(oracle.project(phi, mass, feat), np.float64))
    scale = np.abs(phi * mass[:, None]).T.astype(np.float64) @ np.abs(feat)
    assert np.all(err <= 2e-6 * scale + _floor((phi * mass[:, None]).T, feat, 33))
    if decades == 2:  # within 2^-11 of each other: nothing but the roundings
        assert np.all(err <= 2e-6 * scale)


@pytest.mark.parametrize("decades", [4, 8, 16])
@pytest.mark.parametrize("k", [30, 120, 299])
def test_backward(dev, k, decades):
    """Eigenfunctions apart: basis columns times s_j, rows of dA divided by s_j."""
    import torch
    from paper_2604_10377_amd import fmap as F
    n, d = 211, 140
    rng = np.random.default_rng(decades + k)
    s = _spread(rng, k, decades)
    phi = (rng.standard_normal((n, k)) * s[None, :]).astype(np.float32)
    dA = (rng.standard_normal((k, d)) / s[:, None]).astype(np.float32)
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32)
    dF = F.fmap_project_backward(*(torch.from_numpy(x[None]).to(dev) for x in (phi, mass, dA)))[0].cpu().numpy()
    err = np.abs(dF - np.asarray(oracle.project_backward(phi, mass, dA), np.float64)) / mass[:, None]
    scale = np.abs(phi).astype(np.float64) @ np.abs(dA)
    assert np.all(err <= 1e-6 * scale + _floor(phi, dA, 37))
    if decades == 4:
        assert np.all(err <= 1e-6 * scale)


@pytest.mark.parametrize("decades", [4, 8, 16])
@pytest.mark.parametrize("D", [32, 128, 256])
def test_gradient_features(dev, D, decades):
    """Channels apart under a nearly diagonal A."""
    import torch
    from paper_2604_10377_amd import fmap as F
    V = 133
    rng = np.random.default_rng(decades + D)
    z = (rng.standard_normal((V, D, 2)) * _spread(rng, D, decades)[None, :, None]).astype(np.float32)
    off = 1e-3 * rng.standard_normal((2, D, D))
    Ar, Ai = ((np.diag(rng.standard_normal(D)) + off[i]).astype(np.float32) for i in range(2))
    g = F.fmap_gradient_features(*(torch.from_numpy(a).to(dev) for a in (z, Ar, Ai)), "A").cpu().numpy()
    err = np.abs(g - gf.gradient_features(z, Ar, Ai, "A"))
    mag, w = np.abs(z.astype(np.float64)).sum(2), (np.abs(Ar) + np.abs(Ai)).astype(np.float64).T
    assert np.all(err <= 1e-6 * mag * (mag @ w) + mag * _floor(mag, w, 36))
    if decades == 4:
        assert np.all(err <= 1e-6 * mag * (mag @ w))
