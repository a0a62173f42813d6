"""Backward-weight of fully-connected layers on both sides of the line between the kernels: names, and every element against
64 bits, for sizes with remainders of rows, columns and images.
"""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import host
from net_util import GpuNet
from test_gpu_conv_exact import _logged

pytestmark = pytest.mark.gpu


# images, inputs, outputs, in pieces?  64 blocks of 128 x 128 and 30 000 blocks x images are where the line lies
@pytest.mark.parametrize("B,IN,OUT,pieces", [(470, 1024, 1024, True), (468, 1024, 1024, False), (333, 1111, 1290, True),
                                             (13, 6400, 5900, True), (500, 1020, 777, False), (230, 1500, 1400, True), (230, 1500, 1160, False)])
def test_weight_gradient(B, IN, OUT, pieces):
    rng = np.random.default_rng(B)
    layers = [dict(kind="fc", inputs=[-1], out=OUT), dict(kind="fc", inputs=[0], out=3), dict(kind="softmax_ce", inputs=[1])]
    t = cg_synth.net_tensors(layers, (IN, 1, 1), B, 1, seed=B, num_classes=3)
    t["x"] = rng.standard_normal((B, IN, 1, 1)).astype(np.float32)
    gn = GpuNet(layers, (IN, 1, 1), B, t)
    _, names = _logged(lambda: (gn.step((0.0, 0.0, 0.0, 1.0), cg.CG_STEP_SERIAL), gn.sync()))
    assert any("128x128,rr-,pieces" in n for n in names) == pieces, names
    dy = host(gn.act(0, 1)).reshape(B, OUT).astype(np.float64)
    ref = dy.T @ t["x"].reshape(B, IN).astype(np.float64)
    err = host(gn.g[0])[:OUT * IN].reshape(OUT, IN) - ref
    # B additions in a row, each rounded to nearest, of zero-mean terms: sqrt(B / 6) * 2^-24, and the result's own rounding
    assert np.linalg.norm(err) < ((B / 6) ** 0.5 + 1) * 2.0 ** -24 * np.linalg.norm(ref)
    assert np.abs(err).max() < 2.0 ** -24 * (B + 1) * np.abs(dy).max() * np.abs(t["x"]).max()


def test_outputs_beyond_the_row_tiles_of_the_kernel_in_pieces():
    """65 536 tiles of 128 rows, one more than a launch takes along y: the kernel with taller tiles runs it."""
    B, IN, OUT = 2, 1, 65535 * 128 + 1
    layers = [dict(kind="fc", inputs=[-1], out=OUT), dict(kind="softmax_ce", inputs=[0])]
    t = cg_synth.net_tensors(layers, (IN, 1, 1), B, 1, seed=B, num_classes=OUT)
    gn = GpuNet(layers, (IN, 1, 1), B, t)
    gn.step((0.0, 0.0, 0.0, 1.0), cg.CG_STEP_SERIAL)
    gn.sync()
    dy = host(gn.act(0, 1)).reshape(B, OUT).astype(np.float64)
    ref = (dy * t["x"].reshape(B, 1)).sum(0)
    err = np.abs(host(gn.g[0])[:OUT] - ref)
    # two products and their sum, each rounded to nearest, and half of the smallest subnormal
    assert (err <= 3 * 2.0 ** -24 * np.abs(dy * t["x"].reshape(B, 1)).sum(0) + 2.0 ** -149).all()
