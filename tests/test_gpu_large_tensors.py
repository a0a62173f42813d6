"""Tensors of just under the 2^29 elements a tensor may have, through the kernels that address them in their own way: the first and
the last images, whose byte offsets lie at both ends of 31 bits, on small integers, against 64 bits."""
import pytest
import torch

import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_bwd_weight, conv_fwd
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu
LIMIT = 2 ** 29
F = torch.nn.functional


def _ints(shape, seed):
    return torch.randint(-3, 4, shape, device="cuda", dtype=torch.int8, generator=torch.Generator(device="cuda").manual_seed(seed)).float()


def _ends(t):
    return t[[0, -2, -1]].cpu().double()


# (pass, B, C, H, W, M, k, stride, pad, groups), kernel
CASES = {
    "stem": (("fwd", 3470, 3, 227, 227, 16, 11, 4, 0, 1), "igemm_stem_kernel<"),
    "rectangles_fwd": (("fwd", 1865, 17, 130, 130, 16, 3, 1, 1, 1), "igemm_patch16_kernel<16x128"),
    "rectangles_bwd_data": (("bd", 1865, 16, 130, 130, 17, 3, 1, 1, 1), "igemm_patch16_kernel<16x128"),
    "rectangles_strided": (("bd", 315, 3, 412, 412, 40, 7, 2, 3, 1), "igemm_patch16_kernel<16x128"),
    "a_thread_per_element": (("bd", 64, 8, 1024, 1023, 8, 3, 2, 1, 8), None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_both_ends(name):
    (which, B, C, H, W, M, k, stride, pad, groups), kernel = CASES[name]
    d = cg.conv_desc(B, C, H, W, M, k, stride=stride, pad=pad, groups=groups)
    OH, OW = cg.cg_conv_out_shape(d)
    assert 0.98 * LIMIT < max(B * C * H * W, B * M * OH * OW) < LIMIT
    a, w = _ints((B, C, H, W) if which == "fwd" else (B, M, OH, OW), 1), _ints((M, C // groups, k, k), 2)
    cg.cg_debug_patch_min_tiles(1 if "rectangles" in name else 512)
    try:
        got, names = _logged(lambda: conv_fwd(d, a, w, None) if which == "fwd" else conv_bwd_data(d, a, w))
    finally:
        cg.cg_debug_patch_min_tiles(512)
    assert kernel in names[0] if kernel else not names, names
    if which == "fwd":
        ref = F.conv2d(_ends(a), w.cpu().double(), stride=stride, padding=pad, groups=groups)
    else:
        rest = tuple(n - ((o - 1) * stride - 2 * pad + k) for n, o in ((H, OH), (W, OW)))
        ref = F.conv_transpose2d(_ends(a), w.cpu().double(), stride=stride, padding=pad, output_padding=rest, groups=groups)
    assert torch.equal(_ends(got), ref)
    assert bool(got.isfinite().all())           # (the output was NaN before)


def test_slices_of_the_small_tile_kernel():
    """Backward-weight over 16.7 million pixels: the first and the last pixels of the batch are among the few that count."""
    B, C, H, W, M = 32, 32, 724, 723, 4
    assert 0.98 * LIMIT < B * C * H * W < LIMIT
    x, dy = _ints((B, C, H, W), 3), torch.zeros((B, M, H, W), device="cuda")
    at = [(0, 0, 0, 0), (0, 3, 0, 5), (17, 1, 400, 77), (31, 2, 723, 720), (31, 3, 723, 722), (31, 0, 723, 722)]
    ref = torch.zeros((M, C), dtype=torch.float64)
    for n, m, h, wd in at:
        dy[n, m, h, wd] = 2
        ref[m] += 2 * x[n, :, h, wd].cpu().double()
    (dw, db), names = _logged(lambda: conv_bwd_weight(cg.conv_desc(B, C, H, W, M, 1), x, dy))
    assert names[0].startswith("igemm_direct_kernel<"), names
    assert torch.equal(dw.cpu().double().reshape(M, C), ref) and db.tolist() == [4, 2, 2, 4]
