"""Overlap metrics at the limits of the work split: shapes of one wave (up to 8192 vertices where the mean is
at most 2048), of one workgroup (up to 65536), and longer ones counted in slices by many workgroups next to
short and empty ones; arrays that are not 16-byte aligned.  Counts are integers and the metrics one rounding of
the oracle's float64 arithmetic: compared for equality."""
import numpy as np
import pytest

from oracle import overlap as ov

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [
    [2047, 2049, 2048],
    [8191, 1, 8192, 0, 0, 0, 8193, 7] + [3] * 30,
    [65535, 65536, 65537, 2, 300000],
    [0, 200001, 0, 0] + [5] * 200 + [66000, 0],
    [9000] * 70 + [131072] * 3,
])
@pytest.mark.parametrize("shift", [0, 1])
def test_overlap_split_limits(dev, lens, shift):
    import torch
    from paper_2604_10377_amd import fmap as F
    rng = np.random.default_rng(len(lens) + shift)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    scores = rng.random(n).astype(np.float32)
    scores[::13] = np.nan
    scores[1::17] = 0.5
    truth = (rng.integers(0, 3, n) * 127).astype(np.uint8)  # 0, 127 and 254: any nonzero byte is a label
    print("overlap", lens[:5], "shift", shift, flush=True)
    t = lambda a: torch.from_numpy(np.concatenate([a[:1].repeat(shift), a])).to(dev)[shift:]
    rc, rm = ov.overlap_batch(scores, (truth != 0).astype(np.uint8), off, 0.5)
    ts, tt, to = t(scores), t(truth), torch.from_numpy(off).to(dev)
    for _ in range(2):
        c, m = F.fmap_overlap_metrics(ts, tt, to, 0.5)
        np.testing.assert_array_equal(c.cpu().numpy(), rc)
        np.testing.assert_array_equal(m.cpu().numpy(), rm.astype(np.float32))
