"""The kernel that adds the K slices, on both sides of the slice counts at which its form changes: exact on small integers."""
import pytest

import paper_1706_00095_amd as cg
from test_gpu_conv_exact import _all_three

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,slices", [(1, 2), (2, 4), (3, 6), (7, 14), (8, 16), (19, 38), (20, 40), (33, 66), (64, 128), (300, 480)])
def test_slices_add_up(orc32, B, slices):
    """16x16 planes, one tile of the weight gradient: a slice is 128 pixels, and more where that would be over 512 of them."""
    d, _ = _all_three(orc32, B, dict(C=9, H=16, M=20, k=1, stride=1, pad=0, groups=1), seed=B, fwd=False, bwd_data=False)
    bias = min(B, -(-2048 // 20)) * 20 * 4
    assert (cg.cg_conv_workspace_bytes(d, cg.CG_PASS_BWD_WEIGHT) - bias) // (20 * 9 * 4) == slices
