"""A tuning-cache line written by a plan without items for the general projection kernel (16-byte aligned features) and
read by one of the same signature whose shapes are all on it (features 4 bytes off): the grid it takes fills the chip."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_grid_of_another_plan(dev, tmp_path):
    import torch
    from paper_2604_10377_amd import fmap as F
    n, k, d, cache = 3000, 40, 64, tmp_path / "tune.txt"
    rng = np.random.default_rng(5)
    phi, feat = rng.standard_normal((n, k)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    mass = (rng.uniform(0.5, 1.5, n) / n).astype(np.float32)
    t = lambda a: torch.from_numpy(a).to(dev)
    ev, lam = torch.linspace(0, 40, k, device=dev), torch.full((1,), 0.1, device=dev)
    ref = np.asarray(oracle.project(phi, mass, feat))
    scale = (np.abs(phi) * mass[:, None]).T.astype(np.float64) @ np.abs(feat)
    for shift in (0, 1):
        store = torch.empty(n * d + shift, device=dev)
        f = store[shift:].view(n, d).copy_(t(feat))
        assert f.data_ptr() % 16 == 4 * shift
        pair = dict(phi_x=t(phi), phi_y=t(phi), mass_x=t(mass), mass_y=t(mass), feat_x=f, feat_y=f, evals_x=ev, evals_y=ev,
                    lam=lam)
        plan = F.FmapPlan([pair], backward=False, want_AB=True, tune_cache=cache)
        plan.forward()
        torch.cuda.synchronize()
        # one vertex pair per step of a chunk of at most 2048: sqrt(1024) float32 roundings
        assert (np.abs(plan.A[0].cpu().numpy() - ref) / scale).max() <= 32 * 2.0 ** -24
        tuned = plan.tuning()
        plan.close()
    assert tuned["from_cache"]
    assert tuned["grid"] >= torch.cuda.get_device_properties(dev).multi_processor_count
