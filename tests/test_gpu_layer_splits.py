"""LRN in chunks of every length, fused with its pool and not, and 3x3 pooling at stride 2 of planes too large for LDS, forward and
backward, with padding, odd sides, a rectifier's gate, and two pools whose gradients meet: small nets the oracle runs in full.
"""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import host, max_abs_rel
from net_util import GpuNet
from oracle import net as onet

pytestmark = pytest.mark.gpu
TOL = 1e-3                       # fp32 sums of the layers in between (see the layer tests)


def _check(orc32, layers, in_shape, B, fuse):
    t = cg_synth.net_tensors(layers, in_shape, B, 1, seed=B + in_shape[1], num_classes=4, init="fan_in", peer_std=1e-3)
    cg.cg_debug_fuse_lrn_pool(fuse)
    try:
        gn = GpuNet(layers, in_shape, B, t)
    finally:
        cg.cg_debug_fuse_lrn_pool(1)
    gn.step((0.01, 0.9, 5e-4, 1.0))
    gn.sync()
    buckets = {k: v.copy() for k, v in t["buckets"].items()}
    loss, acts, aux = onet.forward(orc32, layers, t["x"], buckets, t["labels"], t["masks"])
    grads, dact, _ = onet.backward(orc32, layers, t["x"], buckets, t["masks"], acts, aux)
    assert abs(float(host(gn.loss)[0]) - float(loss)) <= TOL * max(1.0, abs(float(loss)))
    for li in range(len(layers) - 1):
        if not gn.fused(li) and layers[li]["kind"] != "concat" and layers[li]["kind"] != "softmax_ce":
            assert max_abs_rel(host(gn.act(li)), acts[li].ravel()) <= TOL, ("activation", li)
    for li, ref in dact.items():
        if li != len(layers) - 1 and not gn.grad_folded(li) and not gn.fused(li):
            assert max_abs_rel(host(gn.act(li, 1)), ref.ravel()) <= TOL, ("gradient", li)
    for li in grads:
        assert max_abs_rel(host(gn.g[li]), grads[li]) <= TOL, ("g_local", li)


# planes of 12 317 (winners and dy in 24 KB, dx not beside them) and 17 685 elements (winners and dy not either), one of odd rows only
@pytest.mark.parametrize("side", [(113, 109), (131, 135), (120, 111)])
@pytest.mark.parametrize("pad", [0, 1, 2])
# who the pools read: both the rectifier (the second one's gradient is added), one the rectifier (behind its gate), one each the
# rectifier and the convolution in front of it (behind the gate and added)
@pytest.mark.parametrize("inputs", [(1, 1), (1,), (1, 0)])
def test_pooling_of_large_planes(orc32, side, pad, inputs):
    pools = [dict(kind="maxpool", inputs=[i], k=3, stride=2, pad=pad) for i in inputs]
    layers = [
        dict(kind="conv", inputs=[-1], M=3, k=3, stride=1, pad=1, groups=1),
        dict(kind="relu", inputs=[0]),
        *pools,
        *([dict(kind="concat", inputs=[2, 3])] if len(pools) == 2 else []),
    ]
    layers += [
        dict(kind="avgpool", inputs=[len(layers) - 1]),
        dict(kind="fc", inputs=[len(layers)], out=4),
        dict(kind="softmax_ce", inputs=[len(layers) + 1]),
    ]
    _check(orc32, layers, (2,) + side, 2, 1)


# channels behind the last whole chunk: of 8, then (50 channels) forward / backward of 8 / 12, 12 / 24, 24 / 24, 24 / 48 and 48 / 48; planes of whole
# groups of four pixels and not; all window sizes
@pytest.mark.parametrize("size,M,side,B", [(5, 77, (12, 11), 2), (3, 13, (9, 9), 1), (5, 6, (8, 8), 3), (7, 50, (10, 7), 2), (5, 50, (56, 54), 70),
                                           (5, 50, (56, 54), 115), (5, 50, (56, 54), 170), (5, 50, (56, 54), 240), (5, 50, (56, 54), 270)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_lrn_chunks(orc32, size, M, side, B, fuse):
    layers = [
        dict(kind="conv", inputs=[-1], M=M, k=1, stride=1, pad=0, groups=1),
        dict(kind="relu", inputs=[0]),
        dict(kind="lrn", inputs=[1], size=size, alpha=1e-2, beta=0.75, kappa=1.0),
        dict(kind="maxpool", inputs=[2], k=3, stride=2, pad=0),
        dict(kind="fc", inputs=[3], out=4),
        dict(kind="softmax_ce", inputs=[4]),
    ]
    _check(orc32, layers, (2,) + side, B, fuse)
