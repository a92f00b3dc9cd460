"""Forward and backward by data where the result has few tiles: the kernel that takes its
operands straight into registers and splits a tile's reduction over the waves, under every
variant it is built in, and the 64 x 128 / 128 x 128 tiles of the staged kernel.  Against the
oracle at the edges: pixel counts around a multiple of 32, channel counts that are no multiple
of a tile, an odd number of channel blocks, filters of any extent, the scattering stores of
the strided backward pass, the split over workgroups.  Bars: gpu_util.assert_close."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv, inputs

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

VARIANTS = {conv.CONV_F32: ["1,1,4", "1,1,8", "2,1,8", "1,2,4", "2,2,4", "1,1,8,3"],
            conv.CONV_BF16: ["1,1,4", "1,1,8", "2,1,8", "2,2,4", "1,1,8,3"]}

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 64, 32, 8, 4, 1, 1, 1, 0),         # one whole tile of 32 pixels
    (1, 40, 36, 11, 3, 1, 1, 1, 0),        # 33 pixels, ragged channels both ways
    (3, 24, 72, 5, 7, 3, 3, 1, 1),         # odd number of channel blocks (bf16), images shorter than a tile
    (2, 20, 68, 6, 9, 3, 3, 2, 1),         # odd number of channel blocks (fp32), classes of a strided backward pass
    (1, 4, 8, 3, 3, 3, 3, 1, 1),           # fewer reduction steps than waves
    (2, 48, 40, 9, 10, 1, 1, 2, 0),        # strided 1x1: zero fill around every stored pixel
    (2, 32, 48, 7, 8, 1, 7, 1, (0, 3)),    # rectangular filter, padding on one axis
    (2, 16, 24, 6, 5, 2, 5, 1, (1, 0)),    # a filter no staged kernel is built for
    (2, 3, 16, 12, 10, 7, 7, 2, 3),        # one channel block in; backward: merged classes, shuffled store
    (1, 512, 96, 7, 7, 3, 3, 1, 1),        # a long reduction
]


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_register_operand_kernel_matches_oracle(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, dO = make_inputs(shape, dtype, layer_id=7)
    fwd, bwd = oracle.fwd(I, Wt, stride, pad), oracle.bwd_data(dO, Wt, H, W, stride, pad)
    ran = 0
    for v in VARIANTS[dtype]:
        monkeypatch.setenv("CONVMI_IGEMM_REG", v)
        L = conv.ConvLayer(*shape, dtype=dtype)
        try:
            for which, kind, kw, ref in ((conv.PASS_FWD, "fwd", dict(I=I, Wt=Wt), fwd),
                                         (conv.PASS_BWD_DATA, "bwd", dict(dO=dO, Wt=Wt), bwd)):
                text, f = conv.conv_describe(L.h, which), v.split(",")
                one = text.startswith("igemm_reg ") and " waves=%s frags=%sx%s " % (f[2], f[0], f[1]) in text
                assert one or len(f) == 4, text  # (a split over workgroups: only where the pass may split)
                ran += one
                assert_close(run_pass(L, kind, **kw), ref, dtype, "%s variant %s" % (kind, v))
        finally:
            L.close()
    assert ran >= len(VARIANTS[dtype]), ran


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
def test_register_operand_kernel_fused_operators(dtype, monkeypatch):
    """Scale, bias, residual (the output buffer itself) and ReLU in the store, and where the
    partial results of a reduction split over workgroups are summed."""
    import torch
    shape = (2, 72, 40, 7, 5, 3, 3, 1, 1)
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, res = make_inputs(shape, dtype, layer_id=8)
    rng = np.random.default_rng(5)
    scale, bias = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.normal(0, 0.2, K).astype(np.float32)
    ref = oracle.fwd(I, Wt, stride, pad).astype(np.float64) * scale[:, None, None] + bias[:, None, None] + res
    ref = np.maximum(ref, 0)
    for v in ["2,2,4", "1,1,8"] + (["1,1,8,2"] if dtype == conv.CONV_F32 else []):
        monkeypatch.setenv("CONVMI_IGEMM_REG", v)
        L = conv.ConvLayer(*shape, dtype=dtype)
        try:
            assert conv.conv_describe(L.h, conv.PASS_FWD).startswith("igemm_reg ")
            L.ws.fill_(0xFF)
            L.set_input(I)
            L.set_weights(Wt)
            L.set_outgrad(res)  # (the residual sits in the output buffer)
            pc = []
            for a in (scale, bias):
                t = torch.zeros(L.info.Kp, dtype=torch.float32, device=L.device)
                t[:K] = torch.from_numpy(a)
                pc.append(t)
            L.fwd_fused(bias=pc[1], residual=L.out_blk, relu=True, scale=pc[0])
            assert_close(L.get_output().float().cpu().numpy(), ref, dtype, "fused, variant " + v)
        finally:
            L.close()


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
def test_register_operand_kernel_keeps_images_apart(dtype, monkeypatch):
    """The upper half of an odd last pair of channel blocks lies in the next image: NaN and
    infinities there must not reach this one."""
    shape = (2, 8 * 3 if dtype == conv.CONV_BF16 else 4 * 3, 32, 5, 6, 3, 3, 1, 1)
    I, Wt, _ = make_inputs(shape, dtype, layer_id=9)
    ref = oracle.fwd(I, Wt, 1, 1)
    I[1] = np.nan
    I[1, :, ::2] = np.inf
    for v in VARIANTS[dtype]:
        monkeypatch.setenv("CONVMI_IGEMM_REG", v)
        L = conv.ConvLayer(*shape, dtype=dtype)
        try:
            got = run_pass(L, "fwd", I=I, Wt=Wt)
        finally:
            L.close()
        assert_close(got[0], ref[0], dtype, "image 0, variant " + v)
        assert np.isnan(got[1]).all()


SMALL_TILES = [  # forward and backward shapes for the 64 x 128 and 128 x 128 tiles, ragged last tiles
    (3, 64, 144, 13, 15, 3, 3, 1, 1), (2, 48, 80, 19, 11, 3, 3, 2, 0), (3, 64, 192, 12, 13, 1, 1, 1, 0),
    (2, 96, 64, 17, 17, 1, 7, 1, (0, 3)), (2, 64, 96, 17, 16, 7, 1, 1, (3, 0)), (2, 48, 64, 20, 21, 5, 5, 1, 2),
    (2, 16, 16, 20, 21, 5, 5, 1, 2),
    (3, 32, 64, 9, 8, 1, 3, 1, (0, 1)), (3, 64, 32, 9, 8, 3, 1, 1, (1, 0)),
]


def _small_tile_exists(shape, dtype, which, fk):
    """Whether the tile is built and fits for this pass: 5x5 filters in bf16 only, the 128-channel tile only where
    one step covers the reduction (two buffers of 25 taps exceed the LDS); the residue classes of a strided
    backward pass on their own in bf16 only."""
    N, C, K, H, W, R, S, stride, pad = shape
    if R == 5:
        return dtype == conv.CONV_BF16 and (fk == 1 or (C if which == "fwd" else K) <= 16)
    return dtype == conv.CONV_BF16 or stride == 1 or which == "fwd"


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SMALL_TILES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_small_staged_tiles_match_oracle(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, dO = make_inputs(shape, dtype, layer_id=10)
    refs = {"fwd": oracle.fwd(I, Wt, stride, pad), "bwd": oracle.bwd_data(dO, Wt, H, W, stride, pad)}
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    monkeypatch.setenv("CONVMI_BWD_QUAD", "0")
    for fk in (1, 2):
        for npl in ((8, 4) if R * S == 1 else (2,)):
            monkeypatch.setenv("CONVMI_IGEMM_CAND", "2,2,%d,2,2,%d" % (fk, npl))
            L = conv.ConvLayer(*shape, dtype=dtype)
            try:
                for which, kind, kw in ((conv.PASS_FWD, "fwd", dict(I=I, Wt=Wt)), (conv.PASS_BWD_DATA, "bwd", dict(dO=dO, Wt=Wt))):
                    text = conv.conv_describe(L.h, which)
                    assert not text.startswith("igemm_reg ")
                    ran = " waves=2x2 frags=%dx2 npl=%d " % (fk, npl) in text
                    assert ran == _small_tile_exists(shape, dtype, kind, fk), text
                    if ran:
                        assert_close(run_pass(L, kind, **kw), refs[kind], dtype, "%s %d %d" % (kind, fk, npl))
            finally:
                L.close()
