"""Weight update on the kernel with small blocks of dW (a filter row per workgroup, the waves split the
pixels, operands through rings of LDS patches), under every variant it is built in, with one split (dW written
directly) and several, against the oracle at the edges: pixel counts around a wave's stage, rows and images
shorter than a run of four pixels, ragged channels both ways, strides, pads per axis, filters of 1, 3, 5 and 7
columns.  Bars: gpu_util.assert_close for an fp32 result."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv, inputs

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

VARIANTS = {1: ["1,1,8,4", "2,2,8,2", "2,4,8,2"], 3: ["1,1,8,2", "1,2,8,2", "2,2,8,2", "2,2,4,4"], 5: ["1,1,8,2"],
            7: ["1,1,8,2"]}

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 32, 32, 1, 1, 1, 1, 1, 0),          # a single pixel
    (3, 72, 136, 5, 5, 1, 1, 1, 0),         # ragged channels, images cross stages
    (2, 264, 40, 12, 11, 1, 1, 1, 0),       # two stages of sixteen pixels per wave and a remainder
    (2, 48, 68, 9, 8, 1, 1, 2, 0),          # strided
    (1, 20, 24, 3, 3, 3, 3, 1, 1),          # every row shorter than a run
    (5, 64, 64, 14, 14, 3, 3, 1, 1),
    (2, 40, 100, 13, 15, 3, 3, 2, 1),       # strided, odd extents
    (3, 36, 32, 11, 9, 3, 3, 2, 0),         # strided, no padding
    (2, 64, 40, 9, 17, 1, 3, 1, (0, 1)),
    (2, 33, 65, 17, 6, 3, 1, 1, (1, 0)),
    (2, 48, 72, 17, 17, 7, 1, 1, (3, 0)),
    (2, 40, 48, 17, 17, 1, 7, 1, (0, 3)),
    (2, 40, 36, 9, 11, 5, 5, 1, 2),         # five columns
    (1, 24, 40, 12, 13, 5, 5, 2, 0),
    (1, 12, 40, 5, 150, 3, 3, 1, 1),        # rows of more than 128 pixels
    (1, 24, 40, 10, 12, 7, 7, 2, 3),        # seven launches' worth of filter rows in one
    (2, 16, 24, 9, 7, 2, 3, 1, (1, 2)),     # an even number of filter rows, more padding than "same"
]


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_ring_update_matches_oracle(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, dtype, layer_id=12)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    for v in VARIANTS[S]:
        for splits in (1, 3):
            monkeypatch.setenv("CONVMI_UPD_RING", "%s,%d" % (v, splits))
            L = conv.ConvLayer(*shape, dtype=dtype)
            try:
                assert conv.conv_describe(L.h, conv.PASS_UPD).startswith("upd_ring ")
                got = run_pass(L, "upd", I=I, dO=dO)
                assert np.isfinite(L.dwt_blk.cpu().numpy()).all()  # (padded channel slots too)
            finally:
                L.close()
            assert_close(got, ref, conv.CONV_F32, "%s splits %d" % (v, splits))


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", [(5, 64, 96, 14, 14, 3, 3, 1, 1), (3, 96, 64, 17, 17, 1, 1, 1, 0)],
                         ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_ring_update_is_exact_on_integers_and_repeatable(shape, dtype, monkeypatch):
    """Small integers: every sum is exact in fp32, so the planner's own choice must match the oracle bit for
    bit, on every call."""
    N, C, K, H, W, R, S, stride, pad = shape
    I = inputs.gen_small_ints((N, C, H, W), -3, 3, which=3)
    dO = inputs.gen_small_ints((N, K, H, W), -3, 3, which=4)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert conv.conv_describe(L.h, conv.PASS_UPD).startswith("upd_ring ")
        for _ in range(3):
            assert np.array_equal(run_pass(L, "upd", I=I, dO=dO), ref.astype(np.float32))
    finally:
        L.close()


@pytest.mark.parametrize("splits", [2, 8, 9, 64, 65, 257])
def test_partial_copies_are_summed_whole(splits, monkeypatch):
    """Numbers of partial copies around those at which the summing kernel changes its number of chains (8, 64)
    and its groups of eight loads; small integers, so that the sums are exact."""
    shape = (1, 20, 24, splits, 128, 3, 3, 1, 1)  # (a copy per row of 128 pixels)
    N, C, K, H, W, R, S, stride, pad = shape
    I = inputs.gen_small_ints((N, C, H, W), -3, 3, which=3)
    dO = inputs.gen_small_ints((N, K, H, W), -3, 3, which=4)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    monkeypatch.setenv("CONVMI_UPD_RING", "1,1,8,2,%d" % splits)
    L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
    try:
        assert "splits=%d " % splits in conv.conv_describe(L.h, conv.PASS_UPD)
        assert np.array_equal(run_pass(L, "upd", I=I, dO=dO), ref.astype(np.float32))
    finally:
        L.close()
