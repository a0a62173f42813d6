"""The kernels that multiply fp32 operands in three bf16 pieces, family by family: every piece of every operand
counts (sums of one product each, 24-bit operands, bit for bit), and rounding is that of fp32 sums, for zero-mean operands
and for operands of one sign; and which of the kernels a problem gets.
"""
import numpy as np
import pytest
import torch

import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_bwd_weight, conv_fwd, dev, host
from net_util import GpuNet
from test_gpu_conv_exact import _logged
from test_gpu_operand_range import _Kernel

import cg_synth

pytestmark = pytest.mark.gpu

FAMILIES = {
    "patch_rows_16": _Kernel("fwd", (3, 32, 13, 16, 3, 1, 1), "igemm_patch16_kernel<16x128,4>", patch=True),
    "patch_rows_32": _Kernel("fwd", (3, 80, 13, 30, 3, 1, 1), "igemm_patch16_kernel<32x128,4>", patch=True),
    "patch_rows_48": _Kernel("fwd", (2, 48, 9, 33, 3, 1, 1), "igemm_patch16_kernel<48x128,4>", patch=True),
    "patch_64": _Kernel("fwd", (4, 48, 13, 200, 3, 1, 1), "igemm_patch_kernel<64x128,4>", patch=True),
    "patch_128": _Kernel("fwd", (9, 32, 13, 128, 3, 1, 1), "igemm_patch_kernel<128x128,4>", patch=True, resident=2),
    "patch_192": _Kernel("fwd", (9, 32, 13, 192, 3, 1, 1), "igemm_patch_kernel<192x128,4>", patch=True, resident=2),
    "patch_192_five_chunks": _Kernel("fwd", (9, 16, 27, 192, 5, 2, 1), "igemm_patch_kernel<192x128,5>", patch=True, resident=2),
    "patch_192_six_chunks": _Kernel("fwd", (2, 16, 56, 192, 3, 1, 1), "igemm_patch_kernel<192x128,6>", patch=True, resident=2),
    "patch_bwd_data": _Kernel("bd", (2, 64, 27, 96, 5, 2, 1), "igemm_patch_kernel<64x128,5>", patch=True),
    "band_64": _Kernel("bw", (4, 24, 14, 64, 5, 2, 1), "igemm_kernel<64x144,band4>", resident=2),
    "band_64_eight_chunks": _Kernel("bw", (2, 40, 90, 64, 3, 1, 1), "igemm_kernel<64x144,band8>", resident=2),
    "band_128": _Kernel("bw", (5, 20, 27, 72, 3, 1, 1), "igemm_kernel<128x144,band8>", resident=2),
    "band_192": _Kernel("bw", (7, 208, 13, 384, 3, 1, 1), "igemm_kernel<192x144,band4>", resident=2),
    "pieces_16": _Kernel("fwd", (76, 20, 34, 8, 3, 0, 1), "igemm_kernel<16x128,4r-,pieces>"),
    "pieces_16_padded": _Kernel("fwd", (80, 21, 33, 13, 3, 1, 1), "igemm_kernel<16x128,4rc,pieces>"),
    "pieces_128": _Kernel("fwd", (53, 29, 24, 113, 3, 0, 1), "igemm_kernel<128x128,4r-,pieces>"),
    "pieces_128_padded": _Kernel("bd", (90, 119, 24, 21, 3, 1, 1), "igemm_kernel<128x128,4rc,pieces>"),
    "pieces_filters_in_place": _Kernel("bd", (25, 512, 14, 32, 1, 0, 1), "igemm_kernel<128x128,rr-,pieces>"),
    "pieces_filters_in_place_four_waves": _Kernel("bd", (100, 320, 14, 99, 1, 0, 1), "igemm_kernel<128x128,rr-,pieces>"),
}


def _one_hot(shape, rng, per):
    """One power of two in every row (per: number of leading axes that make a row), nothing else."""
    t = np.zeros(shape, np.float32)
    rows = t.reshape(int(np.prod(shape[:per])), -1)
    rows[np.arange(len(rows)), rng.integers(0, rows.shape[1], size=len(rows))] = 2.0 ** rng.integers(-9, 10, size=len(rows))
    return t


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("family", list(FAMILIES))
def test_every_piece_of_every_operand_counts(family, swap):
    """One operand has 24 random bits, the other is zero but for powers of two so placed that a sum has one
    product: the result is that operand's value, shifted, bit for bit."""
    k = FAMILIES[family]
    rng = np.random.default_rng(sum(map(ord, family)))
    sa, sb = k.tensors()
    full = lambda s: ((rng.integers(2 ** 23, 2 ** 24, size=s) * 2 - 1) * 2.0 ** -24 * rng.choice([-1, 1], size=s)).astype(np.float32)
    if k.which == "fwd":         # one filter tap per row / one pixel per image
        a, b = (full(sa), _one_hot(sb, rng, 1)) if not swap else (_one_hot(sa, rng, 1), full(sb))
    elif k.which == "bd":        # one row with one tap per input channel / one pixel of dy per image
        if swap:
            a, b = _one_hot(sa, rng, 1), full(sb)
        else:
            a, b = full(sa), np.zeros(sb, np.float32)
            for c in range(sb[1]):
                b[rng.integers(sb[0]), c, rng.integers(sb[2]), rng.integers(sb[3])] = 2.0 ** rng.integers(-9, 10)
    else:                        # one pixel of x (of dy) per channel in the whole batch
        t, other = (sb, sa) if not swap else (sa, sb)
        one = np.zeros(t, np.float32)
        for c in range(t[1]):
            one[rng.integers(t[0]), c, rng.integers(t[2]), rng.integers(t[3])] = 2.0 ** rng.integers(-9, 10)
        a, b = (full(sa), one) if not swap else (one, full(sb))
    ref = k.exact(a, b)
    assert np.array_equal(ref, ref.astype(np.float32)) and np.count_nonzero(ref) > 0
    got = k.run(a, b)
    bad = np.flatnonzero(got != ref)
    assert bad.size == 0, (bad.size, got.ravel()[bad[:4]], ref.ravel()[bad[:4]])


@pytest.mark.parametrize("family", list(FAMILIES))
def test_rounding_of_every_family(family):
    """Relative 2-norm of the error of K-term sums against 64 bits.  K additions in a row, each rounded to nearest
    (errors uniform within 2^-25 to 2^-24 of the sum so far): zero-mean terms, whose sum grows as sqrt(k),
    sqrt(K / 6) * 2^-24; terms of one sign, whose sum grows as k, sqrt(K / 18) * 2^-24; one rounding
    of the result is added.  Terms of one sign may not be off to one side by more than half a last place."""
    k = FAMILIES[family]
    rng = np.random.default_rng(sum(map(ord, family)) + 1)
    sa, sb = k.tensors()
    terms = {"fwd": sb[1] * sb[2] * sb[3], "bd": sa[1] // k.shape[6] * sb[2] * sb[3], "bw": sa[0] * sa[2] * sa[3]}[k.which]
    for a, b, share in ((rng.standard_normal(sa), rng.standard_normal(sb), 6), (rng.uniform(0.5, 1.5, sa), rng.uniform(0.5, 1.5, sb), 18)):
        a, b = a.astype(np.float32), b.astype(np.float32)
        ref = k.exact(a, b)
        err = k.run(a, b) - ref
        rel = np.linalg.norm(err) / np.linalg.norm(ref)
        assert rel < ((terms / share) ** 0.5 + 1) * 2.0 ** -24, (share, rel, terms)
        if share == 18:
            assert abs(err.sum()) < 2.0 ** -25 * ref.sum(), err.sum() / ref.sum()


def test_fully_connected_passes_in_pieces():
    """128-row tiles of aligned quads on both sides (forward) and of rows along the lanes (backward-data), 24-bit operands
    against 64 bits (bounds as above), and the kernels' names."""
    B, rng = 120, np.random.default_rng(3)
    layers = [dict(kind="fc", inputs=[-1], out=1000), dict(kind="fc", inputs=[0], out=1024), dict(kind="fc", inputs=[1], out=3),
              dict(kind="softmax_ce", inputs=[2])]
    in_shape = (512, 1, 1)
    t = cg_synth.net_tensors(layers, in_shape, B, 1, seed=B, num_classes=3)
    t["x"] = rng.standard_normal((B, 512, 1, 1)).astype(np.float32)
    gn = GpuNet(layers, in_shape, B, t)
    _, names = _logged(lambda: (gn.step((0.0, 0.0, 0.0, 1.0), cg.CG_STEP_SERIAL), gn.sync()))
    assert "igemm_kernel<128x128,44-,pieces>" in names and "igemm_kernel<128x128,4r-,pieces>" in names, names
    W0, b0 = (v.astype(np.float64) for v in (t["buckets"][0][:512000].reshape(1000, 512), t["buckets"][0][512000:]))
    ref = t["x"].reshape(B, 512).astype(np.float64) @ W0.T + b0
    err = host(gn.act(0)).reshape(B, 1000) - ref
    assert np.linalg.norm(err) < ((512 / 6) ** 0.5 + 2) * 2.0 ** -24 * np.linalg.norm(ref)
    dy = host(gn.act(1, 1)).reshape(B, 1024).astype(np.float64)
    ref = dy @ t["buckets"][1][:1024000].reshape(1024, 1000).astype(np.float64)
    err = host(gn.act(0, 1)).reshape(B, 1000) - ref
    assert np.linalg.norm(err) < ((1024 / 6) ** 0.5 + 1) * 2.0 ** -24 * np.linalg.norm(ref)


ROUTES = {
    # short and few-block problems, and backward-weight of 1x1 windows, stay with the gathered kernel
    ("fwd", 32, 192, 28, 96, 1, 0, 1): "igemm_kernel<96x128,4r->",
    ("fwd", 32, 480, 14, 64, 1, 0, 1): "igemm_kernel<64x128,4r->",
    ("bw", 32, 192, 28, 96, 1, 0, 1): "igemm_kernel<96x128,4k->",
    ("bd", 32, 192, 28, 96, 1, 0, 1): "igemm_kernel<192x128,rr->",
    # a window of 25 taps in blocks of nine, 98 pixels a unit: more padding than the rows in LDS are worth
    ("bw", 32, 24, 14, 64, 5, 2, 1): "igemm_kernel<64x128,4kc>",
    ("bw", 32, 192, 7, 384, 3, 1, 1): "igemm_kernel<128x128,4kc>",
    ("bw", 64, 384, 13, 384, 3, 1, 2): "igemm_kernel<192x144,band4>",
    # 340 tiles of 64 rows, 3456 indices: cut along K; 510 tiles and 1728: raw rows
    ("bd", 64, 256, 13, 384, 3, 1, 1): "igemm_kernel<256x128,4rc>",
    ("bd", 64, 384, 13, 384, 3, 1, 2): "igemm_patch_kernel<64x128,4>",
}


@pytest.mark.parametrize("route", list(ROUTES), ids=lambda r: "-".join(map(str, r)))
def test_which_kernel_a_problem_gets(route):
    which, B, C, H, M, k, pad, G = route
    d = cg.conv_desc(B, C, H, H, M, k, pad=pad, groups=G)
    OH, OW = cg.cg_conv_out_shape(d)
    x, w, dy = (torch.zeros(s, device="cuda") for s in ((B, C, H, H), (M, C // G, k, k), (B, M, OH, OW)))
    f = {"fwd": lambda: conv_fwd(d, x, w, None), "bd": lambda: conv_bwd_data(d, dy, w), "bw": lambda: conv_bwd_weight(d, x, dy)}[which]
    _, names = _logged(f)
    assert names[0] == ROUTES[route] or ROUTES[route] in names, names
