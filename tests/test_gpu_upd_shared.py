"""bf16 weight updates with both operands staged once for all waves of a workgroup (upd_shared.hip): every block size against the
oracle at the edges of its blocks, rows and stages.  Bars: gpu_util.assert_close (the products are exact, sums in fp32)."""

import numpy as np
import pytest
import torch

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

BF16 = conv.CONV_BF16
# taps, stride class, fragments (C, K), waves (C, K, pixels), pixels of a stage, positions, buffers
VARIANTS = ["1,1,2,2,2,2,2,64,64,3", "1,1,2,2,1,2,4,128,128,3", "1,1,2,4,2,1,4,64,64,3", "1,1,2,4,2,2,2,64,64,3", "1,1,2,4,4,2,1,64,64,2",
            "7,1,1,1,2,4,1,64,128,3", "7,1,1,1,2,2,2,64,128,3", "7,1,1,1,1,2,4,64,128,3", "3,1,1,1,2,2,2,96,128,3", "3,1,1,1,2,2,1,96,128,2",
            "3,1,1,1,1,2,4,64,128,3", "3,2,1,2,2,2,2,96,256,2", "3,2,1,2,1,2,4,64,256,3", "3,2,2,2,1,2,4,64,256,3", "3,2,2,2,2,2,2,32,128,3"]
SHAPES = [  # N, C, K, H, W, R, S, stride, pad: ragged channel blocks, images smaller than a stage, wide rows, strides, taps left over
    (5, 72, 40, 13, 15, 3, 3, 1, 1), (3, 20, 136, 9, 11, 1, 1, 1, 0), (4, 36, 52, 15, 13, 1, 1, 2, 0), (9, 32, 32, 7, 7, 3, 3, 1, 1),
    (3, 64, 80, 17, 17, 1, 7, 1, (0, 3)), (2, 48, 64, 21, 19, 7, 1, 1, (3, 0)), (4, 64, 72, 15, 17, 3, 3, 2, 1), (3, 136, 24, 18, 35, 3, 3, 2, 0),
    (1, 16, 32, 9, 149, 3, 3, 1, 1), (3, 32, 48, 12, 12, 5, 5, 1, 2), (2, 140, 264, 11, 12, 3, 3, 1, 0), (1, 100, 60, 3, 2, 1, 1, 1, 0),
    (2, 24, 40, 14, 12, 1, 3, 1, (0, 1)), (3, 40, 40, 23, 9, 3, 3, 2, 1),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_update_matches_oracle(shape, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, BF16, layer_id=61)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    ran = 0
    for v in VARIANTS:
        for splits in (1, 3):
            monkeypatch.setenv("CONVMI_UPD_SHARED", "%s,%d" % (v, splits))
            L = conv.ConvLayer(*shape, dtype=BF16)
            try:
                if " instead=upd_shared," not in conv.conv_describe(L.h, conv.PASS_UPD):
                    assert not v.startswith("1,"), v  # (one tap fits everywhere)
                    continue
                ran += 1
                print(shape, v, splits, flush=True)
                assert_close(run_pass(L, "upd", I=I, dO=dO), ref, conv.CONV_F32, "%s splits %d" % (v, splits))
                assert np.isfinite(L.dwt_blk.cpu().numpy()).all()
            finally:
                L.close()
    assert ran >= 10, ran  # (every one-column block, each in one range of pixels and in three)


@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[2], SHAPES[4], SHAPES[5], SHAPES[6], SHAPES[7], SHAPES[13]],
                         ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_infinities_stay_in_the_sums_they_belong_to(shape, monkeypatch):
    """Infinite and NaN input values reach the sums of the taps and pixels that read them and no others: not through pixels past the
    end of a row, of the tensor or of a stage, whose dO is zero."""
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, BF16, layer_id=62)
    rng = np.random.default_rng(9)
    for value, (n, y, x) in zip((np.inf, -np.inf, np.nan), ((0, 0, W - 1), (N - 1, H - 1, W - 1), (N - 1, H // 2, 0))):
        I[n, rng.integers(C), y, x] = value
    with np.errstate(invalid="ignore"):
        ref = oracle.upd(I, dO, R, S, stride, pad)
    fine = np.isfinite(ref)
    assert 0 < fine.mean() < 1
    for v in VARIANTS:
        monkeypatch.setenv("CONVMI_UPD_SHARED", v + ",2")
        L = conv.ConvLayer(*shape, dtype=BF16)
        try:
            if " instead=upd_shared," not in conv.conv_describe(L.h, conv.PASS_UPD):
                continue
            got = run_pass(L, "upd", I=I, dO=dO).astype(np.float64)
            assert np.array_equal(np.isfinite(got), fine), v
            assert np.array_equal(got[~fine], ref[~fine], equal_nan=True), v
            assert_close(np.where(fine, got, 0), np.where(fine, ref, 0), conv.CONV_F32, v)
        finally:
            L.close()


# Layers on either side of the lines, and which kernel runs
LINES = [((18, 632, 40, 59, 60, 7, 1, 1, (3, 0)), True), ((27, 504, 284, 23, 21, 1, 7, 1, (0, 3)), True), ((32, 288, 384, 35, 35, 3, 3, 2, 0), True),
         ((92, 288, 384, 35, 35, 3, 3, 2, 0), True), ((8, 288, 384, 35, 35, 3, 3, 2, 0), False), ((28, 128, 128, 28, 28, 3, 3, 1, 1), False),
         ((64, 80, 192, 35, 35, 1, 1, 1, 0), False), ((4, 128, 128, 17, 17, 1, 7, 1, (0, 3)), False)]


@pytest.mark.parametrize("shape,shared", LINES, ids=lambda s: str(s) if isinstance(s, bool) else "x".join(map(str, s)).replace(" ", ""))
def test_chosen_and_as_exact(shape, shared):
    """The plan's choice; where it is this kernel, its error against 64 bits is that of 32-bit sums."""
    N, C, K, H, W, R, S, stride, pad = shape
    L = conv.ConvLayer(*shape, dtype=BF16)
    try:
        assert (" instead=upd_shared," in conv.conv_describe(L.h, conv.PASS_UPD)) == shared
        if not shared:
            return
        I, _, dO = make_inputs(shape, BF16, layer_id=63)
        pads = pad if isinstance(pad, tuple) else (pad, pad)
        x, g = torch.from_numpy(I).double(), torch.from_numpy(dO).double()
        x = torch.nn.functional.pad(x, (pads[1], pads[1], pads[0], pads[0]))
        P, Q = dO.shape[2:]
        flat = g.permute(1, 0, 2, 3).reshape(K, -1)
        got = run_pass(L, "upd", I=I, dO=dO)
        for r, s in {(0, 0), (R - 1, S - 1), (R // 2, S // 2)}:
            v = x[:, :, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].permute(0, 2, 3, 1).reshape(-1, C)
            assert_close(got[:, :, r, s], (flat @ v).numpy(), conv.CONV_F32, "tap %d,%d" % (r, s))
    finally:
        L.close()
