"""Small contractions in one launch (direct_kernel): exact on small integers in every form of operand it takes, at the edges
of its 16 x 32 tiles and of the sixteens of its reduction; and refused for too little workspace as before."""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_weight, conv_fwd, dev, host
from test_gpu_conv_exact import _all_three

pytestmark = pytest.mark.gpu

# (B, C, H, W, M, k, stride, pad, groups): passes that go to the kernel
CASES = {
    "one_of_everything": ((1, 1, 3, 3, 1, 3, 1, 0, 1), "fwd bd bw"),
    "rows_15_columns_31": ((1, 15, 31, 1, 15, 1, 1, 0, 1), "fwd bd bw"),
    "rows_17_columns_33": ((1, 17, 33, 1, 17, 1, 1, 0, 1), "fwd bd bw"),
    "padding_groups": ((3, 26, 7, 9, 34, 3, 1, 1, 2), "fwd bd bw"),
    "long_reduction_16_waves": ((2, 190, 9, 8, 20, 3, 1, 1, 1), "fwd bd"),
    "planes_of_odd_pixels": ((4, 9, 5, 7, 21, 3, 1, 1, 1), "fwd bd bw"),
    "stride_2": ((5, 19, 13, 11, 37, 5, 2, 1, 1), "fwd bd bw"),
    "stride_beyond_window": ((2, 6, 11, 11, 9, 1, 3, 0, 1), "fwd bd bw"),
    "fewer_than_8_rows": ((2, 1, 21, 18, 40, 3, 2, 1, 1), "bd"),
    "fewer_than_8_rows_11x11": ((2, 2, 29, 29, 8, 11, 2, 3, 2), "bd"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_direct_kernel_exact(orc32, name):
    (B, C, H, W, M, k, stride, pad, groups), passes = CASES[name]
    cfg = dict(C=C, H=H, W=W, M=M, k=k, stride=stride, pad=pad, groups=groups)
    for p in passes.split():
        _, names = _all_three(orc32, B, cfg, seed=len(name), fwd=p == "fwd", bwd_data=p == "bd", bwd_weight=p == "bw")
        assert len(names) == 1 and names[0].startswith("igemm_direct_kernel<"), (p, names)


# sums over pixels cut into slices: 1x1 windows at stride 1 (both operands in quads) and others, planes of a multiple of four pixels
# and not, up to 32 columns and few tiles of more
SLICED = [(3, 1, 40, 41, 17, 1, 1, 0, 1), (5, 32, 21, 23, 33, 1, 1, 0, 1), (6, 14, 20, 20, 10, 1, 1, 0, 2), (4, 3, 37, 29, 20, 3, 1, 1, 1), (2, 3, 60, 51, 16, 3, 2, 0, 1),
          (3, 4, 31, 30, 11, 5, 1, 2, 1), (9, 40, 14, 15, 12, 1, 1, 0, 1)]


@pytest.mark.parametrize("case", SLICED, ids=lambda c: "-".join(map(str, c)))
def test_sliced_sums_over_pixels_exact(orc32, case):
    B, C, H, W, M, k, stride, pad, groups = case
    _, names = _all_three(orc32, B, dict(C=C, H=H, W=W, M=M, k=k, stride=stride, pad=pad, groups=groups), seed=C, fwd=False, bwd_data=False)
    # (slices: a workspace for more than the partial sums of the bias gradient)
    assert names in (["igemm_direct_kernel<16x32,44>"], ["igemm_direct_kernel<16x32,4r>"], ["igemm_direct_kernel<16x32,4c>"]), names
    d = cg.conv_desc(B, C, H, W, M, k, stride=stride, pad=pad, groups=groups)
    assert cg.cg_conv_workspace_bytes(d, cg.CG_PASS_BWD_WEIGHT) >= 2 * M * C // groups * k * k * 4


def test_quads_on_both_sides_stop_at_an_image():
    """1x1 windows over 33 pixels an image: what a quad of either operand holds behind an image's last pixel is another channel's."""
    d = cg.conv_desc(40, 5, 3, 11, 6, 1)
    x, dy = torch.ones((40, 5, 3, 11), device="cuda"), torch.ones((40, 6, 3, 11), device="cuda")
    x[:, 2], dy[:, 3] = float("inf"), float("nan")
    dw, db = conv_bwd_weight(d, x, dy)
    dw = dw.reshape(6, 5)
    keep = torch.tensor([[m != 3 and c != 2 for c in range(5)] for m in range(6)], device="cuda")
    assert bool((dw[keep] == 1320).all()) and not bool(dw[~keep].isfinite().any())
    assert bool((db[[0, 1, 2, 4, 5]] == 1320).all()) and bool(db[3].isnan())


def test_what_lies_behind_a_reduction_stays_out():
    """NaN in the next row's first filter values and in the pixels behind an image's last ones: 27 indices and 35 pixels are no
    whole quads, and what a quad holds beyond them belongs to another sum."""
    d = cg.conv_desc(2, 3, 7, 5, 4, 3, pad=1)
    x = torch.ones((2, 3, 7, 5), device="cuda")
    w, dy = torch.ones((4, 3, 3, 3), device="cuda"), torch.ones((2, 4, 7, 5), device="cuda")
    ref = conv_fwd(d, x, w, None).clone()
    w[1] = float("nan")
    y = conv_fwd(d, x, w, None)
    assert torch.equal(y[:, 0], ref[:, 0]) and torch.equal(y[:, 2:], ref[:, 2:]) and bool(y[:, 1].isnan().all())
    rdw, rdb = (t.clone() for t in conv_bwd_weight(d, x, dy))
    dy[0, 1] = float("nan")
    dw, db = conv_bwd_weight(d, x, dy)
    keep = [0, 2, 3]
    assert torch.equal(dw[keep], rdw[keep]) and torch.equal(db[keep], rdb[keep]) and bool(dw[1].isnan().all())


def test_too_little_workspace_is_refused_whichever_kernel_runs():
    d = cg.conv_desc(3, 26, 7, 9, 34, 3, pad=1, groups=2)
    c, x, w, b, dy = cg_synth.conv_layer_int_tensors(dict(C=26, H=7, W=9, M=34, k=3, stride=1, pad=1, groups=2), 3, 1)
    dx = torch.empty((3, 26, 7, 9), device="cuda")
    need = cg.cg_conv_workspace_bytes(d, cg.CG_PASS_BWD_DATA)
    for nbytes in (16, need - 16):
        with pytest.raises(cg.CgError) as e:
            cg.cg_conv_bwd_data(d, dev(dy), dev(w), dx, torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        assert e.value.code == cg.CG_ENOSPC
    assert np.asarray(host(dx)).shape == x.shape
