"""Sums of K slices four columns at a time and one by one: bit for bit on integers, for few and many slices, planes that are whole
groups of four pixels and not, with bias, and accumulated behind a rectifier's gate.
"""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_bwd_weight, conv_fwd, host
from net_util import GpuNet

pytestmark = pytest.mark.gpu


def _ints(rng, *shape):
    return torch.from_numpy(rng.integers(-3, 4, size=shape).astype(np.float32)).cuda()


# 1x1 layers cut along K: images, channels, pixels a side, filters
@pytest.mark.parametrize("B,C,H,M", [(6, 832, 14, 128), (6, 832, 7, 128), (32, 480, 14, 192), (3, 2048, 6, 96), (1, 4096, 10, 70), (2, 1025, 9, 33)])
def test_sliced_1x1_layers(B, C, H, M):
    rng = np.random.default_rng(C + H)
    d = cg.conv_desc(B, C, H, H, M, 1)
    x, w, b, dy = _ints(rng, B, C, H, H), _ints(rng, M, C, 1, 1), _ints(rng, M), _ints(rng, B, M, H, H)
    xd, wd, yd = (t.double().cpu() for t in (x, w, dy))
    f = torch.nn.functional
    assert torch.equal(conv_fwd(d, x, w, b).double().cpu(), f.conv2d(xd, wd, b.double().cpu()))
    assert torch.equal(conv_bwd_data(d, dy, w).double().cpu(), f.conv_transpose2d(yd, wd))
    dw, db = conv_bwd_weight(d, x, dy)
    ref = yd.transpose(0, 1).reshape(M, -1) @ xd.transpose(0, 1).reshape(C, -1).t().contiguous()
    assert torch.equal(dw.double().cpu().view(M, C), ref) and torch.equal(db.double().cpu(), yd.sum((0, 2, 3)))


# windows: columns of dw in whole groups of four (8 * 9, 64 * 9, 512 * 9) and not (7 * 9, 63 * 9), few slices and many; 32 768 elements of dw is
# where four columns a thread begin (57 and 56 rows of 576 columns)
@pytest.mark.parametrize("B,C,H,M", [(2, 8, 30, 24), (2, 7, 30, 24), (40, 8, 56, 40), (40, 7, 56, 40), (2, 64, 30, 57), (2, 64, 30, 56), (40, 64, 30, 57),
                                     (40, 63, 30, 60), (4, 512, 12, 40), (60, 512, 12, 40)])
def test_sliced_weight_gradients(B, C, H, M):
    rng = np.random.default_rng(C + H)
    d = cg.conv_desc(B, C, H, H, M, 3, pad=1)
    x, dy = _ints(rng, B, C, H, H), _ints(rng, B, M, H, H)
    dw, _ = conv_bwd_weight(d, x, dy)
    u = torch.nn.functional.unfold(x.double().cpu(), 3, padding=1)
    ref = sum(dy[n].double().cpu().view(M, -1) @ u[n].t().contiguous() for n in range(B))
    assert torch.equal(dw.double().cpu().view(M, -1), ref)


@pytest.mark.parametrize("side", [14, 7])
def test_accumulated_behind_a_gate(side):
    """Two 1x1 layers read one rectifier: the second one's backward-data is added to the first one's, both behind the gate."""
    layers = [dict(kind="conv", inputs=[-1], M=96, k=1, stride=1, pad=0, groups=1), dict(kind="relu", inputs=[0]),
              dict(kind="conv", inputs=[1], M=512, k=1, stride=1, pad=0, groups=1), dict(kind="conv", inputs=[1], M=640, k=1, stride=1, pad=0, groups=1),
              dict(kind="concat", inputs=[2, 3]), dict(kind="avgpool", inputs=[4]), dict(kind="fc", inputs=[5], out=3), dict(kind="softmax_ce", inputs=[6])]
    t = cg_synth.net_tensors(layers, (8, side, side), 5, 1, seed=side, num_classes=3, init="fan_in", peer_std=1e-3)
    gn = GpuNet(layers, (8, side, side), 5, t)
    gn.step((0.01, 0.9, 5e-4, 1.0))
    gn.sync()
    b = {k: torch.from_numpy(v).double() for k, v in t["buckets"].items()}
    x = torch.from_numpy(t["x"]).double()
    def conv(li, v, M):
        n = b[li].numel() - M
        return torch.nn.functional.conv2d(v, b[li][:n].view(M, -1, 1, 1), b[li][n:])
    h = conv(0, x, 96).relu().requires_grad_(True)
    y = torch.cat([conv(2, h, 512), conv(3, h, 640)], 1).mean((2, 3))
    n = b[6].numel() - 3
    loss = torch.nn.functional.cross_entropy(y @ b[6][:n].view(3, -1).t() + b[6][n:], torch.from_numpy(t["labels"]).long())
    (gh,) = torch.autograd.grad(loss, h)
    ref = torch.einsum("bmhw,bchw->mc", gh * (h > 0), x)
    got = torch.from_numpy(host(gn.g[0]))[:96 * 8].view(96, 8).double()
    assert (got - ref).norm() < 1e-5 * ref.norm()           # sums of 1152 and 245 fp32 terms
