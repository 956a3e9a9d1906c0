"""The vectorized solve with enough pairs that a workgroup forms 64 rows of H instead of 32: n a multiple of 64, just
past one and just short of one, blocks of kx rows that straddle the 64; first, middle and last pair against the oracle
at the tolerance of the other vectorized tests."""
import numpy as np
import pytest

from oracle import vectorized as vz
from paper_2604_10377_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("P,kx,ky", [(1030, 8, 8), (520, 5, 13), (520, 9, 14), (350, 11, 17)])
def test_rows_of_64(dev, P, kx, ky):
    import torch
    from paper_2604_10377_amd import fmap as F
    args = synth.workload_vectorized(P, kx, 4 * kx, ky=ky, lam=1.0, skew=0.3, tag=83)
    print("vectorized", P, kx, ky, flush=True)
    C, info = F.fmap_solve_vectorized(*(torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in args))
    C, info = C.cpu().numpy(), info.cpu().numpy()
    assert (info == 0).all()
    for p in (0, P // 2, P - 1):
        A, B, D1, D2, lam = (a[p] for a in args)
        ref = vz.solve(A, B, D1, D2, float(lam))
        err = np.linalg.norm(C[p] - ref) / np.linalg.norm(ref)
        assert err <= TOL, (p, err)
