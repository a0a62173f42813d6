"""Infinities and NaN in the gradient that a strided convolution's backward-data reads: a stride phase has only some of the
window's taps, the matrix kernels multiply zeros for the rest, and zero times infinity is no part of the sum.  Every kernel that
runs such a pass, on small integers (exact in all arithmetics): each element is what 64-bit sums over the existing taps give.
"""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, dev, host
from net_util import GpuNet
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu
FP32, BF16, X3 = cg.CG_MATH_FP32, cg.CG_MATH_BF16, cg.CG_MATH_BF16X3

# (B, C, H, W, M, k, stride, pad, groups), arithmetics, what the kernel's name holds, thresholds lowered
CASES = {
    "4_rows": ((2, 1, 21, 18, 12, 3, 2, 1, 1), [FP32], None, {}),                  # (a thread per element: no matrix kernel)
    "4_rows_depthwise": ((2, 6, 15, 14, 6, 3, 2, 1, 6), [FP32], None, {}),
    "4_rows_many_channels": ((2, 1, 21, 18, 30, 3, 2, 1, 1), [FP32], "igemm_direct_kernel", {}),
    "phases_without_taps": ((2, 1, 13, 13, 90, 1, 2, 0, 1), [FP32], "igemm_direct_kernel", {}),
    "12_rows": ((2, 3, 21, 18, 12, 3, 2, 1, 1), [FP32], "igemm_direct_kernel", {}),
    "54_rows_without_taps": ((2, 6, 11, 11, 9, 1, 3, 0, 1), [FP32], "igemm_direct_kernel", {}),
    "gathered_12_rows": ((2, 3, 21, 18, 12, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<32x128", {}),
    "gathered_96_rows": ((2, 24, 21, 18, 12, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<", {}),
    "gathered_200_rows": ((2, 50, 33, 40, 12, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<", {}),
    "gathered_fp32": ((32, 3, 256, 255, 40, 3, 2, 1, 1), [FP32], "igemm_kernel<32x128,4rc>", {}),
    "slices_3": ((1, 3, 13, 13, 96, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<32x128", {}),
    "slices_8": ((1, 3, 13, 13, 256, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<32x128", {}),
    "slices_32": ((1, 3, 13, 13, 1024, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<32x128", {}),
    "slices_64": ((1, 3, 13, 13, 2048, 3, 2, 1, 1), [BF16, X3], "igemm_kernel<32x128", {}),
    "pieces_16": ((50, 3, 80, 80, 46, 3, 2, 1, 1), [FP32, BF16, X3], "igemm_kernel<16x128,4rc,pieces", {}),
    "pieces_128": ((32, 27, 79, 79, 60, 3, 2, 1, 1), [FP32], "igemm_kernel<128x128,4rc,pieces", {}),
    "slices_2_pieces_128": ((16, 27, 79, 79, 64, 3, 2, 1, 1), [FP32], "igemm_kernel<128x128,4rc,pieces", {}),
    "patch_48_rows": ((2, 3, 51, 51, 32, 11, 4, 2, 1), [FP32, BF16, X3], "igemm_patch", dict(tiles=1)),
    "patch_32_rows": ((3, 16, 23, 23, 64, 5, 2, 2, 2), [FP32, BF16, X3], "igemm_patch", dict(tiles=1)),
    "patch_192_rows": ((9, 48, 26, 26, 20, 5, 2, 2, 1), [FP32, BF16, X3], "igemm_patch", dict(tiles=1, resident=2)),
    "patch_120_rows_wide": ((1, 30, 40, 260, 17, 5, 2, 2, 1), [FP32, BF16, X3], "igemm_patch", dict(tiles=1)),
}


def _exact(dy, w, H, W, stride, pad, groups):
    k, (OH, OW) = w.shape[2], dy.shape[2:]
    stride, pad = ((v, v) if isinstance(v, int) else v for v in (stride, pad))
    rest = tuple(n - ((o - 1) * s - 2 * p + k) for n, o, s, p in zip((H, W), (OH, OW), stride, pad))
    dy, w = torch.as_tensor(dy).double(), torch.as_tensor(w).double()
    return torch.nn.functional.conv_transpose2d(dy, w, stride=stride, padding=pad, output_padding=rest, groups=groups).numpy()


def _spoil(dy):
    n, c, h, w = dy.shape
    dy[n // 2, c - 1, h - 1, w - 1] = np.nan
    dy[0, min(1, c - 1), h // 2, w // 2] = np.inf
    dy[n - 1, c // 2, 0, 0] = -np.inf


@pytest.mark.parametrize("name,math", [(n, m) for n in CASES for m in CASES[n][1]])
def test_only_windows_that_hold_it(name, math):
    (B, C, H, W, M, k, stride, pad, groups), _, kernel, hooks = CASES[name]
    d = cg.conv_desc(B, C, H, W, M, k, stride=stride, pad=pad, groups=groups)
    OH, OW = cg.cg_conv_out_shape(d)
    rng = np.random.default_rng(len(name))
    dy, w = (rng.integers(1, 4, size=s).astype(np.float32) for s in ((B, M, OH, OW), (M, C // groups, k, k)))
    _spoil(dy)
    cg.cg_debug_patch_min_tiles(hooks.get("tiles", 512))
    cg.cg_debug_resident_blocks(hooks.get("resident", 512))
    before = cg.cg_debug_launch_count()
    try:
        got, names = _logged(lambda: host(conv_bwd_data(d, dev(dy), dev(w), math)))
    finally:
        cg.cg_debug_patch_min_tiles(512)
        cg.cg_debug_resident_blocks(512)
    assert kernel in names[0] if kernel else not names, names
    # the matrix kernel, the copy of the filters before it, the sum of its slices behind it
    assert cg.cg_debug_launch_count() - before == (1 if kernel in (None, "igemm_direct_kernel") else 3 if "slices" in name else 2)
    ref = _exact(dy, w, H, W, stride, pad, groups)
    assert np.isfinite(ref).any() and not np.isfinite(ref).all()
    assert np.array_equal(got, ref, equal_nan=True), np.argwhere(~((got == ref) | (np.isnan(got) & np.isnan(ref))))[:4]


@pytest.mark.parametrize("C,M,math", [(2, 7, FP32), (2, 60, FP32), (6, 7, FP32), (6, 7, BF16), (6, 7, X3)])
@pytest.mark.parametrize("stride,pad", [((1, 3), (0, 2)), ((3, 1), (2, 0)), ((2, 3), (1, 0))])
def test_strides_that_differ(C, M, math, stride, pad):
    H, W, k, groups = 17, 20, 4, 2
    d = cg.cg_conv_desc(2, C, H, W, M * groups, k, k, *stride, *pad, groups)
    rng = np.random.default_rng(C + M)
    dy, w = (rng.integers(1, 4, size=s).astype(np.float32) for s in ((2, M * groups) + tuple(cg.cg_conv_out_shape(d)), (M * groups, C // groups, k, k)))
    _spoil(dy)
    ref = _exact(dy, w, H, W, stride, pad, groups)
    assert np.isfinite(ref).any() and not np.isfinite(ref).all()
    assert np.array_equal(host(conv_bwd_data(d, dev(dy), dev(w), math)), ref, equal_nan=True)


@pytest.mark.parametrize("C,flags", [(4, 0), (4, cg.CG_STEP_BF16X3), (1, 0)])
@pytest.mark.parametrize("branches", [1, 2])
def test_gate_and_accumulation(branches, C, flags):
    """In a net: behind a rectifier, whose gate is applied on the way, and into a gradient that two strided layers share.  The
    infinite gradient comes from weights of the head that add up to 6e38 behind a channel whose output is zero."""
    H, M, OH = 9, 5, 5
    layers = [dict(kind="conv", inputs=[-1], M=C, k=1, stride=1, pad=0, groups=1), dict(kind="relu", inputs=[0])]
    layers += [dict(kind="conv", inputs=[1], M=M, k=3, stride=2, pad=1, groups=1) for _ in range(branches)]
    if branches == 2:
        layers.append(dict(kind="concat", inputs=[2, 3]))
    head = len(layers)
    layers += [dict(kind="fc", inputs=[head - 1], out=2), dict(kind="softmax_ce", inputs=[head])]
    t = cg_synth.net_tensors(layers, (3, H, H), 1, 1, seed=3, num_classes=2)
    t["labels"][:] = 0
    t["buckets"][head][:-2] *= 1e-3
    t["buckets"][head][-2:] = (-50, 50)                 # the wrong class for sure: the logits' gradient is (-1, 1)
    weights = t["buckets"][head][:-2].reshape(2, branches * M, OH, OH)
    for i in range(branches):
        filters, bias = t["buckets"][2 + i][:-M].reshape(M, C, 3, 3), t["buckets"][2 + i][-M:]
        filters[1], bias[1] = 0, 0
        weights[0, M * i + 1, 2, 3 - i], weights[1, M * i + 1, 2, 3 - i] = -3e38, 3e38
    gn = GpuNet(layers, (3, H, H), 1, t)
    gn.step((0.0, 0.0, 0.0, 1.0), flags)
    gn.sync()
    dx = 0.
    for i in range(branches):
        dy = host(gn.act(2 + i, 1)).reshape(1, M, OH, OH)
        assert np.isposinf(dy[0, 1, 2, 3 - i]) and np.isfinite(dy).sum() == dy.size - 1
        dx = dx + _exact(dy, t["buckets"][2 + i][:-M].reshape(M, C, 3, 3), H, H, 2, 1, 1)
    open_gate = host(gn.act(1)).reshape(dx.shape) > 0
    ref, got = np.where(open_gate, dx, 0), host(gn.act(0, 1)).reshape(dx.shape)
    assert not np.isfinite(dx[~open_gate]).all() and not np.isfinite(ref).all()
    ok = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.abs(got[ok] - ref[ok]).max() <= 1e-4 * np.abs(ref[ok]).max()
