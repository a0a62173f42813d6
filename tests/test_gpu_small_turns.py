"""Small nets whose backward-weight passes stay on the compute stream, all of them or some beside others on the third stream: the
overlapped schedule gives the one-stream schedule's bits, step after step."""
import numpy as np
import pytest

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import host
from net_util import GpuNet

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,size", [(4, 12), (64, 40)], ids=["all_small", "small_and_large"])
def test_overlapped_equals_serial(M, size):
    layers = [dict(kind="conv", inputs=[-1], M=M, k=3, stride=1, pad=1, groups=1), dict(kind="relu", inputs=[0]),
              dict(kind="conv", inputs=[1], M=M, k=5, stride=1, pad=2, groups=1), dict(kind="relu", inputs=[2]),
              dict(kind="maxpool", inputs=[3], k=2, stride=2, pad=0), dict(kind="conv", inputs=[4], M=6, k=1, stride=1, pad=0, groups=1),
              dict(kind="fc", inputs=[5], out=7), dict(kind="softmax_ce", inputs=[6])]
    state = []
    for flags in (cg.CG_STEP_SERIAL, cg.CG_STEP_OVERLAP):
        gn = GpuNet(layers, (3, size, size), 5, cg_synth.net_tensors(layers, (3, size, size), 5, 2, seed=4, num_classes=7))
        for _ in range(4):
            gn.step((0.01, 0.9, 5e-4, 1.0), flags)
        gn.sync()
        state.append([host(t).copy() for d in (gn.w, gn.v, gn.g) for t in d.values()])
    assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(*state))
