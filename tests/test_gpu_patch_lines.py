"""Where the patch kernel begins and ends for channels that are no multiple of 16, for windows of four taps and for strided
backward-data, on both sides of each line; and the workspace where one arithmetic takes it and another does not."""
import pytest
import torch

import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_fwd
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu

# (pass, B, C, H, W, M, k, stride, pad): does the patch kernel run it in fp32?
LINES = {
    # strided, up to 48 rows: 265 existing taps times channels, many zeros, and more of the former
    ("bd", 80, 3, 156, 156, 35, 11, 4, 0): False, ("bd", 122, 3, 196, 196, 69, 7, 4, 0): False, ("bd", 13, 12, 136, 136, 18, 11, 2, 0): False,
    ("bd", 86, 4, 121, 91, 137, 7, 3, 0): True, ("bd", 162, 8, 30, 30, 202, 5, 2, 2): True,
    # more than 48 rows and fewer than 500 tiles
    ("bd", 137, 55, 20, 22, 54, 3, 1, 1): False, ("fwd", 10, 26, 31, 35, 269, 5, 1, 2): False, ("fwd", 25, 30, 28, 22, 207, 5, 1, 2): True,
    # forward without padding
    ("fwd", 20, 38, 100, 100, 28, 3, 1, 0): False, ("fwd", 230, 204, 14, 14, 45, 3, 1, 0): True, ("fwd", 183, 104, 56, 56, 59, 2, 1, 0): False,
    # few rows that the small-tile kernel is the faster one for
    ("bd", 133, 12, 20, 20, 124, 3, 1, 1): False, ("bd", 82, 14, 23, 28, 67, 5, 1, 2): True,
}


@pytest.mark.parametrize("line", list(LINES), ids=lambda l: "-".join(map(str, l)))
def test_which_problems_the_patch_kernel_gets(line):
    which, B, C, H, W, M, k, stride, pad = line
    d = cg.conv_desc(B, C, H, W, M, k, stride=stride, pad=pad)
    x, w, y = (torch.zeros(s, device="cuda") for s in ((B, C, H, W), (M, C, k, k), (B, M) + tuple(cg.cg_conv_out_shape(d))))
    _, names = _logged(lambda: conv_fwd(d, x, w, None) if which == "fwd" else conv_bwd_data(d, y, w))
    assert any(n.startswith("igemm_patch") for n in names) == LINES[line], names


@pytest.mark.parametrize("math", [cg.CG_MATH_FP32, cg.CG_MATH_BF16])
def test_workspace_where_only_the_other_arithmetic_takes_it(math):
    """2x2 without padding, 208 -> 32 channels: the gathered kernel in fp32, two K slices of 4 MB; the patch kernel, a copy of
    0.1 MB, in bf16.  What cg_conv_workspace_bytes says is enough for either."""
    d = cg.conv_desc(8, 208, 65, 65, 32, 2)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, w = (torch.randint(-3, 4, s, device="cuda", generator=gen).float() for s in ((8, 208, 65, 65), (32, 208, 2, 2)))
    y, names = _logged(lambda: conv_fwd(d, x, w, None, math))
    assert names[0].startswith("igemm_patch") == (math == cg.CG_MATH_BF16), names
    assert torch.equal(y, torch.nn.functional.conv2d(x.double(), w.double()).float())
