"""The tiled row solve at the edges of its tiles: whole tiles only (the right-hand side in a tile row of its own),
one column and 31 columns in the last tile, three to ten tile columns; and a zero pivot at the ends of the two
16-column halves of a tile, in the first tile, the ones whose update is begun a step ahead, and the last."""
import numpy as np
import pytest

import oracle
from paper_2604_10377_amd import synth

pytestmark = pytest.mark.gpu


def _inputs(seed, P, k):
    rng = synth.rng_for(556, seed, k, k)
    A, B = (rng.standard_normal((P, k, 2 * k)).astype(np.float32) for _ in range(2))
    ex, ey = (np.stack([synth.eigenvalues_linear(rng, k) for _ in range(P)]).astype(np.float32) for _ in range(2))
    return A, B, ex, ey, (10.0 ** rng.uniform(-3, 0, P)).astype(np.float32)


def _solve(dev, args):
    import torch
    from paper_2604_10377_amd import fmap as F
    t = [torch.from_numpy(a).to(dev) for a in args]
    r = [F.fmap_solve(*t, 0, 0.5, store_factors=s) for s in (True, False)]
    torch.cuda.synchronize()
    return [(C.cpu().numpy(), info.cpu().numpy()) for C, _, info, _ in r]


# A A^T has a condition near 30 here (d = 2 k): 1e-5 is its product with the float32 unit roundoff, times five
@pytest.mark.parametrize("k", [66, 95, 97, 128, 129, 159, 160, 192, 193, 256, 257, 287, 288])
def test_tile_edges(dev, k):
    args = _inputs(1, 2, k)
    print("tiled solve k", k, flush=True)
    for C, info in _solve(dev, args):
        assert (info == 0).all()
        for p in range(2):
            ref, rinfo = oracle.solve(args[0][p], args[1][p], oracle.mask(args[2][p], args[3][p], 0, 0.5), float(args[4][p]))
            err = np.linalg.norm(C[p] - ref) / np.linalg.norm(ref)
            assert err <= 1e-5, (p, err)


@pytest.mark.parametrize("k,pivot", [(100, 0), (100, 15), (100, 16), (100, 31), (100, 96), (100, 99), (150, 47), (150, 48),
                                     (150, 64), (150, 149), (300, 33), (300, 95), (300, 207), (300, 272), (300, 288), (300, 299)])
def test_zero_pivot(dev, k, pivot):
    A, B, ex, ey, lam = _inputs(2, 2, k)
    A[0, pivot] = 0.0  # its row and column of the normal matrix are exactly zero
    lam[0] = 0.0
    print("zero pivot", k, pivot, flush=True)
    for C, info in _solve(dev, (A, B, ex, ey, lam)):
        assert (info[0] == pivot + 1).all() and np.isnan(C[0]).all()
        assert (info[1] == 0).all() and np.isfinite(C[1]).all()


@pytest.mark.parametrize("value", [0.0, -1.0, float("nan"), float("inf")])
@pytest.mark.parametrize("k,pivots", [(66, (65,)), (130, (0, 64)), (200, (63, 199)), (200, (64, 127)), (300, (299,))])
def test_bad_stored_pivot(dev, k, pivots, value):
    """The reverse mode with a stored factor reports the first pivot that is not positive and finite, row by row."""
    import torch
    from paper_2604_10377_amd import fmap as F
    A, B, ex, ey, lam = (torch.from_numpy(a).to(dev) for a in _inputs(3, 1, k))
    C, fac, _, _ = F.fmap_solve(A, B, ex, ey, lam, 0, 0.5)
    m, row = k * (k + 1) // 2, k // 2
    for c in pivots:
        fac[0, row * m + c * k - c * (c - 1) // 2] = value
    info = torch.full((1, k), 7, dtype=torch.int32, device=dev)
    print("stored pivot", k, pivots, value, flush=True)
    F.fmap_solve_backward(torch.ones_like(C), A, B, C, ex, ey, lam, 0, 0.5, fac, info=info)
    want = torch.zeros(k, dtype=torch.int32)
    want[row] = pivots[0] + 1
    assert torch.equal(info[0].cpu(), want)
