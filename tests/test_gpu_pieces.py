"""The fp32 contractions multiply in three bf16 pieces per operand on the bf16 matrix instructions: what that
must not change.  Edges of the tiles (row counts around 16, 32, 64, 128; one and two K-slice rounds; eight- and
four-wave blocks; channel counts that leave the patch kernel a last group of 16; odd tap counts), exact on small
integers; rounding against 64 bits; infinities, NaN and values that round to a bf16 infinity."""
import numpy as np
import pytest
import torch

import cg_synth
import paper_1706_00095_amd as cg
from gpu_util import conv_bwd_data, conv_bwd_weight, conv_fwd, dev, host
from test_gpu_conv_exact import _all_three, _descs

pytestmark = pytest.mark.gpu

EDGES = {
    # rows per group around the tile heights; K no multiple of 32; columns no multiple of 128
    "m15": (2, dict(C=5, H=11, M=15, k=3, stride=1, pad=1, groups=1)),
    "m17": (3, dict(C=7, H=9, M=17, k=3, stride=1, pad=0, groups=1)),
    "m33_g2": (2, dict(C=10, H=8, M=66, k=3, stride=1, pad=1, groups=2)),
    "m65": (4, dict(C=13, H=14, M=65, k=1, stride=1, pad=0, groups=1)),
    "m129": (9, dict(C=33, H=14, M=129, k=1, stride=1, pad=0, groups=1)),
    # more than 256 blocks of 128 rows: four-wave blocks
    "four_waves": (24, dict(C=16, H=40, M=128, k=1, stride=1, pad=0, groups=1)),
    "pixels_s2": (5, dict(C=6, H=21, W=18, M=130, k=3, stride=2, pad=1, groups=1)),
}
PATCH = {
    # 48 channels: a group of 32 and one of 16 whose taps go two at a time, the last one alone
    "c48_g1": (2, dict(C=48, H=13, M=72, k=3, stride=1, pad=1, groups=1)),
    "c16_5x5": (1, dict(C=16, H=27, M=200, k=5, stride=1, pad=2, groups=1)),
    "m16": (2, dict(C=32, H=13, M=16, k=3, stride=1, pad=1, groups=1)),
    "m33": (2, dict(C=80, H=9, M=33, k=3, stride=1, pad=1, groups=1)),
}


# backward-weight from padded rows in LDS: several images a unit with the last unit short, bands with a short last
# one, a stride, a channel block that is not full, more than nine taps, row tiles of 64, 128 and 192, slots beyond 256
BANDS = {
    "b13_m384": (7, dict(C=208, H=13, M=384, k=3, stride=1, pad=1, groups=1)),
    "b7_units_of_images": (50, dict(C=44, H=7, M=70, k=3, stride=1, pad=1, groups=1)),
    "b5x5_g2": (5, dict(C=96, H=27, M=136, k=5, stride=1, pad=2, groups=2)),
    "b28_bands": (4, dict(C=64, H=28, W=25, M=64, k=3, stride=1, pad=1, groups=1)),
    "b_stride2_nopad": (6, dict(C=90, H=31, W=29, M=192, k=3, stride=2, pad=0, groups=1)),
    "b_wide": (3, dict(C=40, H=19, W=90, M=64, k=3, stride=1, pad=1, groups=1)),
}


@pytest.mark.parametrize("name", list(BANDS))
def test_band_edges_exact(orc32, name):
    B, cfg = BANDS[name]
    cg.cg_debug_resident_blocks(2)          # a small problem fills a small chip
    try:
        _, names = _all_three(orc32, B, cfg, seed=sum(map(ord, name)), fwd=False, bwd_data=False)
    finally:
        cg.cg_debug_resident_blocks(512)
    assert any(",band" in n for n in names), names


@pytest.mark.parametrize("name", list(EDGES))
def test_tile_edges_exact(orc32, name):
    B, cfg = EDGES[name]
    _all_three(orc32, B, cfg, seed=sum(map(ord, name)))


@pytest.mark.parametrize("name", list(PATCH))
def test_patch_edges_exact(orc32, name):
    B, cfg = PATCH[name]
    cg.cg_debug_patch_min_tiles(1)
    try:
        _, names = _all_three(orc32, B, cfg, seed=sum(map(ord, name)), bwd_weight=False)
    finally:
        cg.cg_debug_patch_min_tiles(512)
    assert any(n.startswith("igemm_patch") for n in names), names


@pytest.mark.parametrize("patch", [False, True])
def test_rounding_is_that_of_fp32_sums(orc64, patch):
    """Relative 2-norm of the error of a K-term sum against 64 bits: at most that of K fp32 additions in a
    row, sqrt(K) * 2^-24 / sqrt(6) with zero-mean terms (the sum grows as sqrt(k) while each of the K roundings
    adds 2^-25 / sqrt(3) .. 2^-24 / sqrt(3) of its present size), plus the final rounding."""
    B, cfg = 2, dict(C=64, H=13, M=96, k=3, stride=1, pad=1, groups=1)
    c, x, w, b, dy = cg_synth.conv_layer_tensors("rounding", B, seed=11, cfg=cfg)
    d, od = _descs(B, c)
    if patch:
        cg.cg_debug_patch_min_tiles(1)
    try:
        got = (host(conv_fwd(d, dev(x), dev(w), None)), host(conv_bwd_data(d, dev(dy), dev(w))),
               host(conv_bwd_weight(d, dev(x), dev(dy))[0]))
    finally:
        cg.cg_debug_patch_min_tiles(512)
    x64, w64, dy64 = (t.astype(np.float64) for t in (x, w, dy))
    ref = (orc64.conv_fwd(od, x64, w64, None), orc64.conv_bwd_data(od, dy64, w64), orc64.conv_bwd_weight(od, x64, dy64)[0])
    for g, r, K in zip(got, ref, (64 * 9, 96 * 9, B * 169)):
        err = np.linalg.norm(g - r) / np.linalg.norm(r)
        assert err < (K ** 0.5 / 6 ** 0.5 + 1) * 2.0 ** -24, (err, K)


def _special(B, C, H, M, k, spots, patch, seed=3):
    rng = np.random.default_rng(seed)
    x = rng.uniform(0.5, 1.5, size=(B, C, H, H)).astype(np.float32)
    w = rng.uniform(0.5, 1.5, size=(M, C, k, k)).astype(np.float32) * np.float32(2.0 ** -8)
    for pos, v in spots:
        x[pos] = v
    d = cg.conv_desc(B, C, H, H, M, k, pad=k // 2)
    if patch:
        cg.cg_debug_patch_min_tiles(1)
    try:
        y = host(conv_fwd(d, dev(x), dev(w), None))
    finally:
        cg.cg_debug_patch_min_tiles(512)
    xt, wt = torch.from_numpy(x).double(), torch.from_numpy(w).double()
    return y, torch.nn.functional.conv2d(xt, wt, padding=k // 2).numpy()


@pytest.mark.parametrize("patch", [False, True])
def test_infinities_and_nan_go_where_they_belong(patch):
    """inf times a filter value is an infinity of the product's sign in every window that sees it, NaN is NaN, and
    no other output is touched (other channels' windows, other images, the pixels of neighbouring lanes)."""
    y, ref = _special(3, 32, 13, 40, 3, [((0, 3, 4, 5), np.inf), ((1, 17, 0, 0), -np.inf), ((2, 31, 12, 12), np.nan)], patch)
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(np.isposinf(y), np.isposinf(ref)) and np.array_equal(np.isneginf(y), np.isneginf(ref))
    ok = np.isfinite(ref)
    assert np.abs(y[ok] - ref[ok]).max() <= 1e-5 * np.abs(ref[ok]).max()


@pytest.mark.parametrize("patch", [False, True])
def test_values_beyond_the_largest_bf16_stay_finite(patch):
    """3.3961e38 and up round to a bf16 infinity but are finite fp32 numbers."""
    big = np.float32(3.4e38)
    y, ref = _special(2, 32, 13, 24, 3, [((0, 5, 6, 6), big), ((1, 9, 3, 3), -np.finfo(np.float32).max)], patch)
    assert np.isfinite(y).all()
    assert np.abs(y - ref).max() <= 1e-6 * np.abs(ref).max()
    far = np.abs(ref) < 1e30
    assert np.abs(y[far] - ref[far]).max() <= 1e-5 * np.abs(ref[far]).max()


def test_infinity_in_a_filter_and_in_a_gradient():
    B, C, H, M = 2, 24, 9, 20
    rng = np.random.default_rng(5)
    x, w, dy = (rng.uniform(0.5, 1.5, size=s).astype(np.float32) for s in ((B, C, H, H), (M, C, 3, 3), (B, M, H, H)))
    w[4, 7, 1, 1] = np.inf
    d = cg.conv_desc(B, C, H, H, M, 3, pad=1)
    y = host(conv_fwd(d, dev(x), dev(w), None))
    assert np.isposinf(y[:, 4]).all() and np.isfinite(np.delete(y, 4, axis=1)).all()
    dy[1, 3, 2, 2] = -np.inf
    w[4, 7, 1, 1] = 1.0
    dw, db = (host(t) for t in conv_bwd_weight(d, dev(x), dev(dy)))
    assert np.isneginf(dw[3]).all() and np.isneginf(db[3])
    assert np.isfinite(np.delete(dw, 3, axis=0)).all() and np.isfinite(np.delete(db, 3)).all()
