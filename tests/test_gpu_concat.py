"""The backward of a channel concat, all slices in one launch: slices behind a folded rectifier and without one, of a layer that
also feeds another (its gradient is added to), of a layer that is concatenated twice, and of the net's input, which wants no
gradient; planes and channel counts that can and cannot be moved in fours.  Whole iterations against the oracle."""
import pytest

import cg_synth
from test_gpu_fullsize import _check_step

pytestmark = pytest.mark.gpu


def _conv(src, M, k=1):
    return dict(kind="conv", inputs=[src], M=M, k=k, stride=1, pad=k // 2, groups=1)


def _relu(src):
    return dict(kind="relu", inputs=[src])


# four branches; the second one's rectifier also feeds a convolution behind the concat
def _branches(M):
    layers = [_conv(-1, M[0], 3), _relu(0), _conv(1, M[1]), _relu(2), _conv(1, M[2], 3), _conv(1, M[3]), _relu(5),
              dict(kind="concat", inputs=[3, 4, 6, 1])]
    layers += [_conv(7, 6), _conv(3, 6), dict(kind="concat", inputs=[8, 9])]
    return layers


def _twice(M):
    return [_conv(-1, M[0], 3), _relu(0), _conv(1, M[1]), dict(kind="concat", inputs=[2, 1, 2, -1]), _conv(3, 5)]


@pytest.mark.parametrize("net", [_branches, _twice], ids=["branches", "twice"])
@pytest.mark.parametrize("M,C,size,B", [((8, 16, 4, 12), 4, 7, 3), ((3, 5, 1, 7), 3, 7, 5), ((6, 2, 9, 3), 1, 1, 2),
                                        ((12, 33, 8, 20), 4, 20, 1)],
                         ids=["fours", "odd", "one_pixel", "blocks"])
def test_concat_gradient(orc32, net, M, C, size, B):
    layers = net(M)
    layers += [dict(kind="fc", inputs=[len(layers) - 1], out=7), dict(kind="softmax_ce", inputs=[len(layers)])]
    t = cg_synth.net_tensors(layers, (C, size, size), B, 1, seed=11, num_classes=7, init="fan_in", peer_std=1e-3)
    _check_step(orc32, layers, (C, size, size), B, t)
