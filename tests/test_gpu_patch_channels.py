"""The patch kernel on channel counts that are no multiple of 16, on windows of four taps and on planes so wide that a block takes
a rectangle of pixels: exact on small integers, also in the bf16 modes; what lies behind the last channel stays out; a workspace without room for the padded filter copy."""
import pytest
import torch

import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_fwd
from test_gpu_conv_exact import _all_three, _logged

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def patch_path():
    cg.cg_debug_patch_min_tiles(1)
    yield
    cg.cg_debug_patch_min_tiles(512)


# (B, C, H, W, M, k, stride, pad, groups)
CASES = [
    (3, 1, 13, 13, 17, 3, 1, 1, 1), (2, 15, 13, 11, 72, 3, 1, 0, 1), (2, 17, 13, 13, 130, 3, 1, 1, 1), (3, 31, 9, 9, 33, 3, 1, 2, 1),
    (2, 33, 13, 13, 47, 5, 1, 2, 1), (2, 58, 13, 13, 50, 3, 1, 1, 2), (3, 19, 15, 15, 21, 3, 2, 1, 1), (1, 3, 30, 30, 20, 7, 2, 3, 1),
    (2, 20, 14, 13, 70, 2, 1, 0, 1), (5, 47, 27, 27, 16, 5, 1, 2, 1),
]
# planes whose rows do not fit: rectangles with remainders on both sides, every width the slots allow, groups
WIDE = [(2, 18, 9, 130, 20, 3, 1, 1, 1), (1, 16, 70, 97, 40, 5, 1, 2, 1), (2, 34, 33, 81, 70, 7, 1, 3, 2), (1, 3, 150, 151, 33, 11, 2, 5, 1),
        (1, 16, 65, 129, 130, 3, 1, 0, 1), (1, 21, 127, 3, 17, 3, 1, 1, 1)]


@pytest.mark.parametrize("math", [cg.CG_MATH_FP32, cg.CG_MATH_BF16, cg.CG_MATH_BF16X3])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_any_number_of_channels_exact(orc32, case, math):
    B, C, H, W, M, k, stride, pad, groups = case
    cfg = dict(C=C, H=H, W=W, M=M, k=k, stride=stride, pad=pad, groups=groups)
    _, names = _all_three(orc32, B, cfg, seed=C, bwd_weight=False, math=math)
    assert len([n for n in names if "igemm_patch" in n]) >= (1 if C == 3 else 2), names


@pytest.mark.parametrize("math", [cg.CG_MATH_FP32, cg.CG_MATH_BF16X3])
@pytest.mark.parametrize("case", WIDE, ids=lambda c: "-".join(map(str, c)))
def test_rectangles_of_wide_planes_exact(orc32, case, math):
    test_any_number_of_channels_exact(orc32, case, math)


def test_an_infinity_in_a_rectangle():
    """Infinite exactly where a window reaches it: the sums done again in fp32 find the same pixels."""
    d = cg.conv_desc(1, 17, 40, 130, 20, 3, pad=1)
    x, w = torch.ones((1, 17, 40, 130), device="cuda"), torch.ones((20, 17, 3, 3), device="cuda")
    x[0, 16, 21, 77] = float("inf")
    y, names = _logged(lambda: conv_fwd(d, x, w, None))
    assert any("igemm_patch" in n for n in names), names
    assert bool((~y.isfinite()).nonzero()[:, 2:].unique(dim=0).eq(torch.cartesian_prod(torch.arange(20, 23), torch.arange(76, 79)).cuda()).all())
    assert bool((y[0, :, 20:23, 76:79] == float("inf")).all()) and bool((y[0, :, 1:19, 1:129] == 153).all())


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_the_next_groups_channels_stay_out(value):
    """Five channels a group: the eleven that fill up the sixteen are the next group's, the next image's or nothing."""
    d = cg.conv_desc(2, 10, 13, 13, 14, 3, pad=1, groups=2)
    x, w = torch.ones((2, 10, 13, 13), device="cuda"), torch.ones((14, 5, 3, 3), device="cuda")
    (ref, names) = _logged(lambda: conv_fwd(d, x, w, None).clone())
    assert any("igemm_patch" in n for n in names), names
    x[:, 5:] = value
    y = conv_fwd(d, x, w, None)
    assert torch.equal(y[:, :7], ref[:, :7]) and not bool(y[:, 7:].isfinite().any())
    dy = torch.ones((2, 14, 13, 13), device="cuda")
    ref = conv_bwd_data(d, dy, w).clone()
    dy[:, 7:] = value
    dx = conv_bwd_data(d, dy, w)
    assert torch.equal(dx[:, :5], ref[:, :5]) and not bool(dx[:, 5:].isfinite().any())


@pytest.mark.parametrize("which", ["fwd", "bd", "bd_strided"])
def test_workspace_of_the_other_kernels_is_enough(which):
    """What the gathered kernel needs was enough before the padded copies were made, and still is."""
    stride = 2 if which == "bd_strided" else 1
    d = cg.conv_desc(1, 19, 10, 10, 17, 5, stride=stride, pad=1)
    OH, OW = cg.cg_conv_out_shape(d)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, w, dy = (torch.randint(-3, 4, s, device="cuda", generator=gen).float() for s in ((1, 19, 10, 10), (17, 19, 5, 5), (1, 17, OH, OW)))
    run = (lambda y, ws: cg.cg_conv_fwd(d, x, w, None, y, ws)) if which == "fwd" else (lambda y, ws: cg.cg_conv_bwd_data(d, dy, w, y, ws))
    out = torch.empty_like(dy if which == "fwd" else x)
    p = cg.CG_PASS_FWD if which == "fwd" else cg.CG_PASS_BWD_DATA
    need = cg.cg_conv_workspace_bytes(d, p)
    _, names = _logged(lambda: run(out, torch.empty(need, dtype=torch.uint8, device="cuda")))
    assert any("igemm_patch" in n for n in names), names
    ref = out.clone()
    cg.cg_debug_patch_min_tiles(512)
    less = cg.cg_conv_workspace_bytes(d, p)
    assert less < need
    cg.cg_debug_patch_min_tiles(1)
    out.fill_(float("nan"))
    _, names = _logged(lambda: run(out, torch.empty(less, dtype=torch.uint8, device="cuda")))
    assert not any("igemm_patch" in n for n in names), names
    assert torch.equal(out, ref)
