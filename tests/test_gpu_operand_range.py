"""Operands anywhere in the range of fp32: what three bf16 pieces per operand have to carry, through every kernel
that cuts operands.  Subnormal and nearly subnormal values keep all their bits, products just below 2^128 are
finite, an infinity times a subnormal is an infinity, and an infinity or a NaN of one channel stays out of the others.
"""
import numpy as np
import pytest
import torch

import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_bwd_weight, conv_fwd, dev, host
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu


class _Kernel:
    """A shape, the pass that is looked at, what steers the shape to the kernel, and the kernel's name."""

    def __init__(self, which, shape, name, patch=False, resident=None):
        self.which, self.shape, self.name, self.patch, self.resident = which, shape, name, patch, resident

    def run(self, a, b, math=None):
        """fwd: a = x, b = w; bd: a = dy, b = w; bw: a = dy, b = x."""
        d = self.desc()
        if self.patch:
            cg.cg_debug_patch_min_tiles(1)
        if self.resident:
            cg.cg_debug_resident_blocks(self.resident)
        try:
            f = {"fwd": lambda: conv_fwd(d, dev(a), dev(b), None, math), "bd": lambda: conv_bwd_data(d, dev(a), dev(b), math),
                 "bw": lambda: conv_bwd_weight(d, dev(b), dev(a), math)[0]}[self.which]
            out, names = _logged(lambda: host(f()))
        finally:
            cg.cg_debug_patch_min_tiles(512)
            cg.cg_debug_resident_blocks(512)
        assert any(self.name in n for n in names), names
        return out

    def desc(self):
        B, C, H, M, k, pad, G = self.shape
        return cg.conv_desc(B, C, H, H, M, k, pad=pad, groups=G)

    def tensors(self):
        """Shapes of a and b."""
        B, C, H, M, k, pad, G = self.shape
        OH = H + 2 * pad - k + 1
        x, w, dy = (B, C, H, H), (M, C // G, k, k), (B, M, OH, OH)
        return {"fwd": (x, w), "bd": (dy, w), "bw": (dy, x)}[self.which]

    def exact(self, a, b):
        """The same in 64 bits (0 * inf and 0 * nan are NaN, at padding too)."""
        B, C, H, M, k, pad, G = self.shape
        a, b = torch.from_numpy(a).double(), torch.from_numpy(b).double()
        F = torch.nn.functional
        if self.which == "fwd":
            return F.conv2d(a, b, padding=pad, groups=G).numpy()
        if self.which == "bd":
            return F.conv_transpose2d(a, b, padding=pad, groups=G).numpy()
        u = F.unfold(b, k, padding=pad).view(B, G, C // G * k * k, -1)
        dy = a.reshape(B, G, M // G, -1)
        return torch.stack([sum(dy[n, g] @ u[n, g].t().contiguous() for n in range(B)) for g in range(G)]).reshape(
            M, C // G, k, k).numpy()


KERNELS = {
    "patch_rows_shared": _Kernel("fwd", (2, 48, 9, 33, 3, 1, 1), "igemm_patch16_kernel<48x128,4>", patch=True),
    "patch_64": _Kernel("fwd", (2, 16, 13, 72, 3, 1, 1), "igemm_patch_kernel<64x128,4>", patch=True),
    "patch_bwd_data": _Kernel("bd", (1, 64, 27, 32, 5, 2, 1), "igemm_patch_kernel<64x128,5>", patch=True),
    "band_64": _Kernel("bw", (4, 24, 14, 64, 5, 2, 1), "igemm_kernel<64x144,band4>", resident=2),
    "band_128": _Kernel("bw", (5, 20, 27, 72, 3, 1, 1), "igemm_kernel<128x144,band8>", resident=2),
    "pieces_16": _Kernel("fwd", (76, 20, 34, 8, 3, 0, 1), "igemm_kernel<16x128,4r-,pieces>"),
    "pieces_128": _Kernel("fwd", (53, 29, 24, 113, 3, 0, 1), "igemm_kernel<128x128,4r-,pieces>"),
    "pieces_filters_in_place": _Kernel("bd", (25, 512, 14, 32, 1, 0, 1), "igemm_kernel<128x128,rr-,pieces>"),
}


def _one_per_reduction(shape, rng, scale):
    """Filters (or inputs) with few non-zeros, so that sums are a handful of products."""
    t = np.zeros(shape, np.float32)
    flat = t.reshape(shape[0], -1)
    for r in range(shape[0]):
        c = rng.integers(0, flat.shape[1], size=3)
        flat[r, c] = (rng.uniform(1, 2, size=3) * scale).astype(np.float32)
    return t


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("ea,eb", [(-140, 100), (-149, 120), (-125, 40), (-60, -68), (62.9, 63), (90, -100)])
def test_products_of_extreme_operands(kernel, ea, eb):
    """a around 2^ea times a few b around 2^eb: at most 3 * B products a sum, so fp32 multiply-adds are within
    (products + 1) * 2^-24 of the exact sum (plus half of the smallest subnormal); results beyond 2^128 are infinite on both sides."""
    k = KERNELS[kernel]
    rng = np.random.default_rng(sum(map(ord, kernel)))
    sa, sb = k.tensors()
    a = (rng.uniform(1, 2, size=sa) * 2.0 ** ea).astype(np.float32)
    if k.which == "bw":          # few non-zero pixels of x: as many products a sum
        b = np.zeros(sb, np.float32)
        b[0, :, sb[2] // 2, sb[3] // 2] = rng.uniform(1, 2, size=sb[1]) * 2.0 ** (eb - 1)
    else:
        b = _one_per_reduction(sb, rng, 2.0 ** (eb - 1))
    if k.which == "bd":          # a column of the filters adds up over all rows
        b[1:] = 0
    ref = k.exact(a, b)
    got = k.run(a, b)
    fits = np.abs(ref) < 2.0 ** 127.9
    assert fits.any() and np.isfinite(got[fits]).all()
    bound = 5 * 2.0 ** -24 * np.abs(ref[fits]) + 2.0 ** -149
    assert (np.abs(got[fits] - ref[fits]) <= bound).all(), np.max(np.abs(got[fits] - ref[fits]) / np.maximum(np.abs(ref[fits]), 2.0 ** -149))


@pytest.mark.parametrize("kernel", list(KERNELS))
def test_infinities_and_nan(kernel):
    """One infinity of each sign and one NaN among positive operands, subnormal ones among them (an infinity times
    2^-140 is an infinity), all others finite: every output is what 64-bit arithmetic gives, finite ones as near as fp32
    sums of one sign are (K * 2^-24)."""
    k = KERNELS[kernel]
    rng = np.random.default_rng(9)
    sa, sb = k.tensors()
    a, b = (rng.uniform(0.5, 1.5, size=s).astype(np.float32) for s in (sa, sb))
    tiny = rng.integers(0, b.size, size=b.size // 8)
    b.reshape(-1)[tiny] = np.float32(2.0 ** -140)
    n, c, h, w = sa
    a[0, 1, h // 2, w // 2] = np.inf
    a[n - 1, c // 2, 0, 0] = -np.inf
    a[n // 2, c - 1, h - 1, w - 1] = np.nan
    ref, got = k.exact(a, b), k.run(a, b)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref)
    terms = {"fwd": sb[1] * sb[2] * sb[3], "bd": sa[1] * sb[2] * sb[3], "bw": sa[0] * sa[2] * sa[3]}[k.which]
    assert ok.any() and (np.abs(got[ok] - ref[ok]) <= terms * 2.0 ** -24 * np.abs(ref[ok])).all()


@pytest.mark.parametrize("math", [cg.CG_MATH_FP32, cg.CG_MATH_BF16, cg.CG_MATH_BF16X3])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_weight_gradient_of_other_channels_stays_clean(math, value):
    """14x14 in two bands of 98 pixels: a band's last group of four reaches two pixels beyond it, into the next
    band or the next channel.  What is there must not reach this channel's sums: rows of dw other than the poisoned channel's
    are the same bits as without it."""
    k = _Kernel("bw", (4, 24, 14, 64, 5, 2, 1), "band4", resident=2)
    rng = np.random.default_rng(4)
    sa, sb = k.tensors()
    dy, x = (rng.uniform(0.5, 1.5, size=s).astype(np.float32) for s in (sa, sb))
    clean = k.run(dy, x, math)
    dy[1, 7, 0, 0] = dy[2, 7, 0, 1] = value              # the first pixels of channel 7: behind channel 6's last band
    got = k.run(dy, x, math)
    others = np.arange(64) != 7
    assert np.isfinite(got[others]).all() and np.array_equal(got[others], clean[others])
    assert not np.isfinite(got[7]).any()
    if math == cg.CG_MATH_FP32 and not np.isnan(value):
        # an infinity of its own channel, first pixel of the second band: infinite wherever its window has a pixel of x
        dy[1, 7, 0, 0] = dy[2, 7, 0, 1] = 1
        dy[3, 7, 7, 5] = value
        got = k.run(dy, x, math)
        assert np.array_equal(got[7], np.full_like(got[7], value))


def test_weight_gradient_with_the_scratch_memory_of_the_gathered_kernel():
    """The kernel with rows in LDS cuts this reduction into more slices than the gathered one's 79: a caller that brings
    what that one needs (its slices, and the bias sums of 41 images behind them) gets its result."""
    d = cg.conv_desc(41, 42, 20, 20, 48, 3, pad=1)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, dy = (torch.randint(-3, 4, (41, c, 20, 20), device="cuda", generator=gen).float() for c in (42, 48))
    (ref, rdb), names = _logged(lambda: conv_bwd_weight(d, x, dy))
    assert any("band" in n for n in names), names
    need = -(-79 * 48 * 42 * 9 * 4 // 256) * 256 + 41 * 48 * 4
    assert need < cg.cg_conv_workspace_bytes(d, cg.CG_PASS_BWD_WEIGHT)
    dw, db = torch.full_like(ref, float("nan")), torch.full_like(rdb, float("nan"))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    _, names = _logged(lambda: cg.cg_conv_bwd_weight(d, x, dy, dw, db, ws))
    assert names and not any("band" in n for n in names), names
    assert torch.equal(dw, ref) and torch.equal(db, rdb)
    with pytest.raises(cg.CgError):
        cg.cg_conv_bwd_weight(d, x, dy, dw, db, ws[:-16])
