"""Operands anywhere in the range of fp32, through the kernels that cut operands in bf16 pieces: an infinity or a NaN of
one channel stays out of the others.
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
