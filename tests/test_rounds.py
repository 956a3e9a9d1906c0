"""The chunks of the tall forward projection (64 < k, read from the workspace it asks for): with three column blocks of a
chunk on one of the 8 XCDs, no XCD gets more workgroups than it has CUs where the whole launch is meant as one round.
k and n are no multiples of 4, so that no other kernel's chunks size the workspace.  Without a GPU the library takes
256 CUs."""
import pytest

from paper_2604_10377_amd import fmap as F


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 7, 10, 13, 20])
@pytest.mark.parametrize("n", [5001, 9999, 20001])
@pytest.mark.parametrize("k,d", [(131, 300), (203, 352), (301, 384)])
def test_one_round(batch, n, k, d):
    chunks = F.fmap_project_workspace_bytes(batch, n, k, d) // (4 * batch * k * d)
    each, blocks = 256 // 8, 3  # CUs of an XCD; 128 columns per block for these d
    if batch * chunks * blocks <= 256:
        assert -(-batch * chunks // 8) * blocks <= each


@pytest.mark.parametrize("batch,n,k,d", [(8, 5001, 101, 300), (4, 20001, 127, 352), (10, 9999, 70, 384)])
def test_wide_blocks_fill_the_chip(batch, n, k, d):
    """Up to k = 128, d above 128 is cut into blocks of 256 columns: two for these."""
    chunks = F.fmap_project_workspace_bytes(batch, n, k, d) // (4 * batch * k * d)
    assert 0.9 * 256 <= 2 * batch * chunks <= 2 * 256
