"""Survivor lists where the list's workgroups change from sixteenths to quarters
of a count block and from quarters to whole ones, sparse and with every pair
passing, against the set bits of the mask (whole numbers: equal)."""
import pytest

from tests.test_gpu_survivor_blocks import BLOCK, test_block_edges as block_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pairs", [127 * BLOCK + 8191, 128 * BLOCK - 8192, 128 * BLOCK,
                                     130 * BLOCK + 8193, 511 * BLOCK + 1, 512 * BLOCK + 31])
@pytest.mark.parametrize("density", [0.002, 1.0])
def test_quarter_edges(n_pairs, density):
    block_edges(n_pairs, density)
