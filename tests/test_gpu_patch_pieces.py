"""Patch kernel with three pieces of each filter value in its copy (a workspace with room for them) against fp32 values that it
cuts itself (a workspace of what cg_conv_workspace_bytes says): the same pieces, products and order of sums, so the same bits, in
every row tile and patch size, for ragged channels, groups, strides, and for values outside the pieces' range.
"""
import numpy as np
import pytest
import torch

import paper_1706_00095_amd as cg
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu

# pass, (B, C, H, M, k, stride, pad, groups), resident blocks, kernel
SHAPES = [
    ("fwd", (3, 32, 13, 16, 3, 1, 1, 1), 512, "igemm_patch16_kernel<16x128,4>"),
    ("fwd", (3, 80, 13, 30, 3, 1, 1, 1), 512, "igemm_patch16_kernel<32x128,4>"),
    ("bd", (2, 44, 27, 120, 5, 1, 2, 1), 512, "igemm_patch16_kernel<48x128,5>"),
    ("fwd", (4, 48, 13, 200, 3, 1, 1, 1), 512, "igemm_patch_kernel<64x128,4>"),
    ("fwd", (9, 35, 13, 128, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,4>"),      # groups of 32 and 3 channels
    ("bd", (9, 100, 13, 144, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,4>"),
    ("fwd", (9, 32, 13, 192, 3, 1, 1, 1), 2, "igemm_patch_kernel<192x128,4>"),      # one group of channels
    ("bd", (9, 192, 13, 112, 3, 1, 1, 1), 2, "igemm_patch_kernel<192x128,4>"),      # the octets go round
    ("fwd", (9, 320, 13, 384, 2, 1, 0, 2), 2, "igemm_patch_kernel<192x128,4>"),     # groups of four steps
    ("fwd", (9, 16, 27, 192, 5, 1, 2, 1), 2, "igemm_patch_kernel<192x128,5>"),
    ("fwd", (2, 16, 56, 128, 3, 1, 1, 1), 2, "igemm_patch_kernel<128x128,6>"),
    ("bd", (2, 5, 33, 40, 5, 2, 1, 1), 512, "igemm_patch16_kernel<32x128"),         # (channel, phase) rows
    ("bd", (3, 20, 33, 40, 3, 2, 1, 1), 512, "igemm_patch_kernel<64x128"),
]


@pytest.mark.parametrize("values", ["normal", "range", "inputs"])
@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "-".join(map(str, (c[0],) + c[1])))
def test_pieces_beforehand_or_in_registers(case, values):
    which, (B, C, H, M, k, stride, pad, G), resident, name = case
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
    copy = max(M * ((C // G + 15) // 16 * 16), C * stride * stride * ((M // G + 15) // 16 * 16)) * (k + stride) ** 2 * 6
    outs = []
    cg.cg_debug_patch_min_tiles(1)
    cg.cg_debug_resident_blocks(resident)
    try:
        need = cg.cg_conv_workspace_bytes(d, p)
        padded = (M if which == "fwd" else C) * (((C if which == "fwd" else M) // G + 15) // 16 * 16) * k * k * 4
        for room in (min(need, (padded + 255) // 256 * 256) if stride == 1 else need, need + copy):
            out = torch.full(t["dy" if which == "fwd" else "x"].shape, float("nan"), device="cuda")
            ws = torch.full((max(room, 16),), 255, dtype=torch.uint8, device="cuda")
            run = (lambda: cg.cg_conv_fwd(d, t["x"], t["w"], None, out, ws)) if which == "fwd" else (lambda: cg.cg_conv_bwd_data(d, t["dy"], t["w"], out, ws))
            _, names = _logged(run)
            assert any(name in n for n in names), names
            outs.append(out)
            # the copy ends where the values, or the pieces, of this layout do: three pieces were written where they have room
            if stride == 1:
                torch.cuda.synchronize()
                third = ws[padded:padded * 3 // 2]
                wants = resident != 2 or not name.startswith("igemm_patch_kernel<192x128,5")
                assert (room > need) == bool(third.numel() and (third != 255).any()) or not wants
    finally:
        cg.cg_debug_patch_min_tiles(512)
        cg.cg_debug_resident_blocks(512)
    a, b = (o.view(torch.int32) for o in outs)
    both_nan = outs[0].isnan() & outs[1].isnan()
    assert bool(((a == b) | both_nan).all()), int((~((a == b) | both_nan)).sum())
    if values == "normal":
        f = torch.nn.functional
        x, w, dy = (t[n].double().cpu() for n in ("x", "w", "dy"))
        if which == "fwd":
            ref = f.conv2d(x, w, stride=stride, padding=pad, groups=G)
        else:
            over = H - ((OH - 1) * stride + k - 2 * pad)
            ref = f.conv_transpose2d(dy, w, stride=stride, padding=pad, groups=G, output_padding=over)
        terms = (C if which == "fwd" else M) // G * k * k
        err = (outs[1].double().cpu() - ref).norm() / ref.norm()
        assert err < ((terms / 6) ** 0.5 + 1) * 2.0 ** -24, err       # K roundings of a zero-mean sum
