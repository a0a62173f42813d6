"""Patch kernel with three pieces of each filter value in its copy (a workspace with room for them) against fp32 values that it
cuts itself (a workspace of the size of the values): the same pieces, products and order of sums, so the same bits, in
every row tile and patch size, for ragged channels, groups, strides, and for values outside the pieces' range.
"""
import numpy as np
import pytest
import torch

import paper_1706_00095_amd as cg
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu

# pass, (B, C, H, M, k, stride, pad, groups), resident blocks, kernel, does a workspace with room hold pieces?
SHAPES = [
    ("fwd", (3, 32, 13, 16, 3, 1, 1, 1), 512, "igemm_patch16_kernel<16x128,4>", True),
    ("fwd", (3, 80, 13, 30, 3, 1, 1, 1), 512, "igemm_patch16_kernel<32x128,4>", True),
    ("bd", (2, 44, 27, 120, 5, 1, 2, 1), 512, "igemm_patch16_kernel<48x128,5>", True),
    ("bd", (4, 96, 13, 160, 3, 1, 1, 2), 512, "igemm_patch16_kernel<48x128,4>", True),
    ("fwd", (4, 48, 13, 200, 3, 1, 1, 1), 512, "igemm_patch_kernel<64x128,4>", False),     # less than a round of blocks
    ("fwd", (9, 64, 13, 64, 3, 1, 1, 1), 8, "igemm_patch_kernel<64x128,4>", True),         # one and a half
    ("fwd", (9, 64, 13, 64, 3, 1, 1, 1), 7, "igemm_patch_kernel<64x128,4>", False),        # up to two
    ("fwd", (9, 64, 13, 64, 3, 1, 1, 1), 2, "igemm_patch_kernel<64x128,4>", True),         # six
    ("fwd", (9, 48, 13, 64, 3, 1, 1, 1), 2, "igemm_patch_kernel<64x128,4>", False),        # 432 indices
    ("fwd", (9, 35, 13, 128, 3, 1, 1, 1), 24, "igemm_patch_kernel<128x128,4>", True),      # groups of 32 and 3 channels
    ("fwd", (9, 35, 13, 128, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,4>", False),      # a round and a few blocks
    ("fwd", (64, 35, 13, 128, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,4>", True),      # a second launch for the rest of many rounds
    ("fwd", (9, 32, 13, 128, 3, 1, 1, 1), 24, "igemm_patch_kernel<128x128,4>", False),     # one group of channels
    ("bd", (9, 100, 13, 144, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,4>", True),
    ("bd", (9, 200, 13, 96, 3, 1, 1, 2), 48, "igemm_patch_kernel<128x128,4>", True),       # two groups of filters
    ("fwd", (9, 32, 13, 192, 3, 1, 1, 1), 2, "igemm_patch_kernel<192x128,4>", True),       # one group of channels
    ("bd", (9, 192, 13, 112, 3, 1, 1, 1), 2, "igemm_patch_kernel<192x128,4>", True),       # the octets go round
    ("fwd", (9, 320, 13, 384, 2, 1, 0, 2), 2, "igemm_patch_kernel<192x128,4>", True),      # groups of four steps
    ("fwd", (9, 16, 27, 192, 5, 1, 2, 1), 2, "igemm_patch_kernel<192x128,5>", False),
    ("fwd", (2, 16, 56, 128, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,6>", True),
    ("bd", (2, 5, 33, 40, 5, 2, 1, 1), 512, "igemm_patch16_kernel<32x128", True),          # (channel, phase) rows
    ("bd", (3, 20, 33, 40, 3, 2, 1, 1), 512, "igemm_patch_kernel<64x128", True),
    ("bd", (3, 32, 33, 40, 3, 2, 1, 1), 14, "igemm_patch_kernel<128x128,4>", False),
    ("bd", (2, 10, 33, 48, 5, 2, 1, 2), 512, "igemm_patch16_kernel<32x128", True),         # of two groups
]


def _reference(which, x, w, dy, H, OH, k, stride, pad, G):
    f = torch.nn.functional
    if which == "fwd":
        return f.conv2d(x, w, stride=stride, padding=pad, groups=G)
    return f.conv_transpose2d(dy, w, stride=stride, padding=pad, groups=G, output_padding=H - ((OH - 1) * stride + k - 2 * pad))


@pytest.mark.parametrize("values", ["normal", "range", "inputs"])
@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "-".join(map(str, (c[0],) + c[1] + (c[2],))))
def test_pieces_beforehand_or_in_registers(case, values):
    which, (B, C, H, M, k, stride, pad, G), resident, name, pieces = case
    d = cg.conv_desc(B, C, H, H, M, k, stride=stride, pad=pad, groups=G)
    OH, OW = cg.cg_conv_out_shape(d)
    rng = np.random.default_rng(sum(case[1]))
    t = {n: rng.standard_normal(s).astype(np.float32) for n, s in (("x", (B, C, H, H)), ("w", (M, C // G, k, k)), ("dy", (B, M, OH, OW)))}
    if values == "range":           # filters whose scaled pieces overflow, subnormals, an infinity, a NaN
        w = t["w"].reshape(-1)
        at = rng.permutation(w.size)
        w[at[:4]] = [3e38, 2.0 ** 104, -1.5e-44, 1e-40]
        w[at[4]], w[at[5]] = np.inf, np.nan
    if values == "inputs":          # sums done again from filters of the whole range, subnormal ones and 2^104 and more among them
        t["w"] = (t["w"] * 2.0 ** rng.integers(-140, 106, size=t["w"].shape)).astype(np.float32)
        src = t["x" if which == "fwd" else "dy"]
        src[0, 0], src[-1, -1, 0, 0], src[-1, 1, -1, -1] = np.inf, np.nan, -np.inf
    t = {n: torch.from_numpy(v).cuda() for n, v in t.items()}
    p = cg.CG_PASS_FWD if which == "fwd" else cg.CG_PASS_BWD_DATA
    # bytes of the copy in fp32, half as much again in pieces: rows, channels of a reduction in units of 16, taps
    taps = ((k + stride - 1) // stride) ** 2
    rows, red = (M, C // G) if which == "fwd" else (C * stride * stride, M // G)
    fp32 = rows * ((red + 15) // 16 * 16) * taps * 4
    need = cg.cg_conv_workspace_bytes(d, p)
    outs = []
    cg.cg_debug_patch_min_tiles(1)
    cg.cg_debug_resident_blocks(resident)
    try:
        for room in ((fp32 + 255) // 256 * 256, max(need, fp32 // 2 * 3)):
            out = torch.full(t["dy" if which == "fwd" else "x"].shape, float("nan"), device="cuda")
            ws = torch.full((max(need, fp32 * 2),), 255, dtype=torch.uint8, device="cuda")
            run = (lambda: cg.cg_conv_fwd(d, t["x"], t["w"], None, out, ws[:room])) if which == "fwd" else (lambda: cg.cg_conv_bwd_data(d, t["dy"], t["w"], out, ws[:room]))
            _, names = _logged(run)
            assert any(name in n for n in names), names
            outs.append(out)
            # the copy ends where the values, or the pieces, of this layout do
            written = bool((ws[fp32:fp32 // 2 * 3] != 255).any())
            assert written == (pieces and room >= fp32 // 2 * 3)
            assert bool((ws[fp32 // 2 * 3:] == 255).all())
    finally:
        cg.cg_debug_patch_min_tiles(512)
        cg.cg_debug_resident_blocks(512)
    a, b = (o.view(torch.int32) for o in outs)
    both_nan = outs[0].isnan() & outs[1].isnan()
    assert bool(((a == b) | both_nan).all()), int((~((a == b) | both_nan)).sum())
    x, w, dy = (t[n].double().cpu() for n in ("x", "w", "dy"))
    terms = (C if which == "fwd" else M) // G * k * k
    got = outs[1].double().cpu()
    if values == "normal":
        ref = _reference(which, x, w, dy, H, OH, k, stride, pad, G)
        err = (got - ref).norm() / ref.norm()
        assert err < ((terms / 6) ** 0.5 + 1) * 2.0 ** -24, err       # K roundings of a zero-mean sum
    elif values == "inputs" or which == "fwd":      # (backward-data multiplies infinite filters by the zeros around dy, the reference does not)
        ref = _reference(which, x, w, dy, H, OH, k, stride, pad, G)
        for of in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(of(got), of(ref.float())), of.__name__
        ok = ref.float().isfinite()
        size = _reference(which, *(v.abs().nan_to_num(0, 0, 0) for v in (x, w, dy)), H, OH, k, stride, pad, G)
        # a rounding or a dropped product per term, at most half of the smallest subnormal each at the lower end
        assert ok.any() and bool(((got - ref).abs()[ok] <= (terms + 2) * (2.0 ** -24 * size[ok] + 2.0 ** -149)).all())


# pass, (B, C, H, M, k, stride, pad, groups): a grouped 5x5 layer, ragged channels, a strided one
@pytest.mark.parametrize("which,shape", [("bd", (32, 96, 27, 256, 5, 1, 2, 2)), ("fwd", (44, 70, 27, 48, 5, 1, 2, 1)), ("bd", (64, 12, 55, 48, 5, 2, 2, 1))])
def test_half_as_much_again_as_reported_holds_pieces(which, shape):
    B, C, H, M, k, stride, pad, G = shape
    d = cg.conv_desc(B, C, H, H, M, k, stride=stride, pad=pad, groups=G)
    OH, OW = cg.cg_conv_out_shape(d)
    x, w, y = (torch.ones(s, device="cuda") for s in ((B, C, H, H), (M, C // G, k, k), (B, M, OH, OW)))
    need = cg.cg_conv_workspace_bytes(d, cg.CG_PASS_FWD if which == "fwd" else cg.CG_PASS_BWD_DATA)
    rows, red = (M, C // G) if which == "fwd" else (C * stride * stride, M // G)
    fp32 = rows * ((red + 15) // 16 * 16) * ((k + stride - 1) // stride) ** 2 * 4
    ws = torch.full((need // 2 * 3,), 255, dtype=torch.uint8, device="cuda")
    _, names = _logged(lambda: cg.cg_conv_fwd(d, x, w, None, y, ws) if which == "fwd" else cg.cg_conv_bwd_data(d, y, w, x, ws))
    assert all("igemm_patch" in n for n in names), names
    assert bool((ws[fp32:fp32 // 2 * 3] != 255).any())
