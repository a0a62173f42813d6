"""Forward convolutions of few input channels from rows in LDS: exact on small integers over strides (one, two or four shifted
copies of the rows), window widths around multiples of four, row tiles, groups and planes with remainders on both sides; what
lies beside a window stays out; a workspace without room for the cut filters; a net with such a first layer."""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import conv_fwd, dev, host
from net_util import GpuNet
from test_gpu_conv_exact import _all_three, _logged

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def few_resident_blocks():
    cg.cg_debug_resident_blocks(2)           # small problems are then many rounds of blocks, as large ones are on the GPU
    yield
    cg.cg_debug_resident_blocks(512)


# (B, C, H, W, M, k, stride, pad, groups): row tiles 16, 32, 48, 64, 96, 128 and remainders
CASES = [
    (2, 3, 67, 67, 96, 11, 4, 0, 1), (1, 3, 64, 75, 64, 7, 2, 3, 1), (3, 4, 50, 41, 16, 11, 2, 5, 1), (1, 1, 70, 58, 45, 7, 2, 3, 1),
    (3, 4, 63, 47, 30, 11, 4, 2, 1), (1, 6, 51, 66, 100, 7, 2, 0, 2), (1, 3, 90, 131, 140, 11, 2, 0, 1), (1, 2, 64, 200, 50, 12, 3, 1, 1),
    (2, 3, 40, 40, 33, 11, 1, 5, 1),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_forward_exact(orc32, case):
    B, C, H, W, M, k, stride, pad, groups = case
    _, names = _all_three(orc32, B, dict(C=C, H=H, W=W, M=M, k=k, stride=stride, pad=pad, groups=groups), seed=M, bwd_data=False, bwd_weight=False)
    assert len(names) == 1 and names[0].startswith("igemm_stem_kernel<"), names


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 2.0 ** 120])
def test_what_lies_beside_a_window_stays_out(value):
    """The fourth column of an 11-column window's last quad is a neighbour's pixel; the sums it could spoil are done again."""
    d = cg.conv_desc(1, 3, 67, 67, 64, 11, stride=4)
    x, w = torch.ones((1, 3, 67, 67), device="cuda"), torch.ones((64, 3, 11, 11), device="cuda")
    x[0, 1, 30, 31] = value
    y, names = _logged(lambda: conv_fwd(d, x, w, None))
    assert names[0].startswith("igemm_stem_kernel<"), names
    hit = torch.zeros((15, 15), dtype=torch.bool)
    hit[[r for r in range(15) if 4 * r <= 30 < 4 * r + 11]] = True
    hit &= torch.tensor([4 * c <= 31 < 4 * c + 11 for c in range(15)])
    plain = y[0, :, ~hit.cuda()]
    assert bool((plain == 363).all())
    spoilt = y[0, :, hit.cuda()]
    assert bool((spoilt == value).all()) if value == value else bool(spoilt.isnan().all())


def test_accuracy_and_workspace():
    """24-bit operands against 64 bits: 2 roundings of 2^-24 a value and about sqrt(steps) / 2 of the sum; without room for the cut
    filters the gathered kernel's result, the fp32 instruction's."""
    d = cg.conv_desc(2, 1, 67, 67, 96, 11, stride=4)
    c, x, w, b, dy = cg_synth.conv_layer_tensors("stem", 2, seed=5, cfg=dict(C=1, H=67, M=96, k=11, stride=4, pad=0, groups=1))
    ref = torch.nn.functional.conv2d(torch.tensor(x).double(), torch.tensor(w).double(), torch.tensor(b).double(), stride=4).numpy()
    err = np.linalg.norm(host(conv_fwd(d, dev(x), dev(w), dev(b))) - ref) / np.linalg.norm(ref)
    assert err < 2 * 2.0 ** -24, err
    y = torch.full((2, 96, 15, 15), float("nan"), device="cuda")
    ws = torch.empty(max(16, cg.cg_conv_workspace_bytes(d, cg.CG_PASS_FWD) - 16), dtype=torch.uint8, device="cuda")
    _, names = _logged(lambda: cg.cg_conv_fwd(d, dev(x), dev(w), dev(b), y, ws))
    assert not any("stem" in n for n in names), names
    assert np.linalg.norm(host(y) - ref) / np.linalg.norm(ref) < 121 ** 0.5 * 2.0 ** -24


def test_in_a_net(orc32):
    """Filters cut with the other layers' copies at the start of an iteration, the rectifier folded into the store."""
    layers = [dict(kind="conv", inputs=[-1], M=20, k=7, stride=2, pad=3, groups=1), dict(kind="relu", inputs=[0]),
              dict(kind="fc", inputs=[1], out=5), dict(kind="softmax_ce", inputs=[2])]
    t = cg_synth.net_tensors(layers, (3, 40, 36), 4, 1, seed=2, num_classes=5)
    t["x"] = np.random.default_rng(1).integers(-3, 4, size=(4, 3, 40, 36)).astype(np.float32)
    t["buckets"][0] = np.random.default_rng(2).integers(-3, 4, size=20 * 147 + 20).astype(np.float32)
    gn = GpuNet(layers, (3, 40, 36), 4, t)
    _, names = _logged(lambda: (gn.step((0.0, 0.0, 0.0, 1.0)), gn.sync()))
    assert any("igemm_stem_kernel" in n for n in names), names
    ref = torch.nn.functional.conv2d(torch.tensor(t["x"]).double(), torch.tensor(t["buckets"][0][:2940].reshape(20, 3, 7, 7)).double(),
                                     torch.tensor(t["buckets"][0][2940:]).double(), stride=2, padding=3).clamp(min=0).numpy()
    assert np.array_equal(host(gn.act(1)).reshape(ref.shape), ref)
