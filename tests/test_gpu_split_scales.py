"""The scales of the split forward projections (float32): rows and columns that are zero in the first stage of 32
vertices of a chunk, or in the one where another value outgrows its scale, and are then far smaller than the others;
infinities beside them; vertices without mass.  220 vertices are one chunk of seven stages in every kernel.

Tolerance, per entry: the two-part products keep 22 bits of each operand, the general float32 routine 24, and either
sums at most 110 steps in float32: a few 2^-24 sqrt(steps) of the sum of the entry's terms' magnitudes, 2e-6.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 2e-6
N = 220
# k <= 64 (three widths of its basis windows), then one size for each instance of the tall kernel
SIZES = [(30, 128), (45, 300), (64, 512), (70, 128), (122, 300), (150, 260), (250, 320), (319, 400)]


def _inputs(k, d, kind):
    rng = np.random.default_rng(1000 + k)
    mass = rng.uniform(0.5, 1.5, N) / N
    phi, feat = rng.standard_normal((N, k)), rng.standard_normal((N, d))
    late = slice(32, None)
    if kind.startswith("late column"):
        feat[:32, 5] = 0
        feat[late, 5] *= float(kind.split()[-1])
    elif kind.startswith("late row"):
        phi[:32, 5] = 0
        phi[late, 5] *= float(kind.split()[-1])
    elif kind == "zero where a column outgrows":
        feat[64:96, 5] = 0
        feat[70, 3] = 1e10
    elif kind == "zero where a row outgrows":
        phi[64:96, 5] = 0
        phi[70, 3] = 1e10
    elif kind == "zero until a column has outgrown":
        feat[:96, 5] = 0
        feat[96:, 5] *= 1e-3
        feat[70, 3] = 1e10
    elif kind == "infinite feature":
        feat[:96, 5] = 0
        feat[70, 3] = np.inf
    elif kind == "infinite basis value":
        phi[:96, 5] = 0
        phi[70, 3] = np.inf
    elif kind == "no mass":
        mass[10] = 0
        feat[10] = 1e8
    elif kind == "no mass beside a late column":
        mass[10] = mass[40] = 0
        feat[:32, 5] = 0
        feat[late, 5] *= 1e-8
        feat[10, 5] = feat[40, 5] = 1
    return phi.astype(np.float32), mass.astype(np.float32), feat.astype(np.float32)


KINDS = ["late column 1e-6", "late column 1e-10", "late column 1e-30", "late row 1e-6", "late row 1e-10", "late row 1e-30",
         "zero where a column outgrows", "zero where a row outgrows", "zero until a column has outgrown",
         "infinite feature", "infinite basis value", "no mass", "no mass beside a late column"]


def _check(A, phi, mass, feat):
    if np.isinf(feat).any():
        assert np.array_equal(A[:, 3], np.sign(phi[70]) * np.inf)
        A, feat = np.delete(A, 3, 1), np.delete(feat, 3, 1)
    if np.isinf(phi).any():
        assert np.array_equal(A[3], np.where(feat[70] != 0, np.sign(feat[70]) * np.inf, np.nan), equal_nan=True)
        A, phi = np.delete(A, 3, 0), np.delete(phi, 3, 1)
    scale = (np.abs(phi).astype(np.float64) * mass[:, None]).T @ np.abs(feat).astype(np.float64)
    err = np.abs(A - np.asarray(oracle.project(phi, mass, feat), np.float64))
    assert (err / scale).max() <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("k,d", SIZES)
def test_every_row_and_column_keeps_its_bits(dev, k, d, kind):
    import torch
    from paper_2604_10377_amd import fmap as F
    arrays = _inputs(k, d, kind)
    A = F.fmap_project(*(torch.from_numpy(x).to(dev)[None] for x in arrays))[0].cpu().numpy()
    _check(A, *arrays)


@pytest.mark.parametrize("kind", ["late column 1e-10", "late row 1e-10", "zero where a column outgrows",
                                  "infinite feature", "no mass beside a late column"])
def test_plan(dev, kind):
    import torch
    from paper_2604_10377_amd import fmap as F
    pairs, arrays = [], []
    for k in (45, 120):
        phi, mass, feat = _inputs(k, 256, kind)
        arrays.append((phi, mass, feat))
        t = [torch.from_numpy(x).to(dev) for x in (phi, mass, feat)]
        ev = torch.linspace(0, 30, k, device=dev)
        pairs.append(dict(phi_x=t[0], phi_y=t[0], mass_x=t[1], mass_y=t[1], feat_x=t[2], feat_y=t[2], evals_x=ev,
                          evals_y=ev, lam=torch.full((1,), 0.1, device=dev)))
    plan = F.FmapPlan(pairs, backward=False, want_AB=True)
    plan.forward()
    torch.cuda.synchronize()
    for i in range(2):
        _check(plan.A[i].cpu().numpy(), *arrays[i])
        _check(plan.B[i].cpu().numpy(), *arrays[i])
    plan.close()
