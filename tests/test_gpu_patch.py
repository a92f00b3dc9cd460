"""Forward and backward by data on the kernel with a tile's pixels in LDS (bf16, filters of seven and nine taps), under
every variant it is built in, against the oracle at its edges: tiles that cross rows and images, images smaller
than a tile, ragged channels (an odd number of channel blocks, fewer blocks than waves), strides, pads other
than "same", the longest patch.  Bars: gpu_util.assert_close."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

VARIANTS = ["1,1,8", "2,1,8", "1,2,8", "2,2,4", "2,2,8", "1,2,4", "2,4,4", "1,4,4", "1,4,8"]

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 8, 8, 1, 1, 3, 3, 1, 1),            # a single pixel, a single channel block
    (5, 72, 40, 7, 7, 3, 3, 1, 1),          # images smaller than a tile, an odd number of channel blocks
    (3, 64, 136, 13, 15, 3, 3, 1, 1),
    (1, 280, 24, 9, 8, 3, 3, 1, 1),         # two and three pairs of channel blocks to a wave
    (2, 40, 48, 6, 52, 3, 3, 1, 1),         # long rows
    (2, 24, 40, 12, 11, 3, 3, 1, 0),        # no padding: rows of the result are shorter than the input's
    (2, 40, 36, 8, 9, 3, 3, 2, 1),          # strided
    (3, 48, 72, 17, 17, 1, 7, 1, (0, 3)),
    (3, 48, 72, 9, 11, 7, 1, 1, (3, 0)),
    (2, 24, 40, 6, 9, 3, 3, 1, (0, 1)),     # padding on one axis
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_patch_kernel_matches_oracle(shape, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, dO = make_inputs(shape, conv.CONV_BF16, layer_id=9)
    cases = [("fwd", conv.PASS_FWD, dict(I=I, Wt=Wt), oracle.fwd(I, Wt, stride, pad))]
    if stride == 1:
        cases.append(("bwd", conv.PASS_BWD_DATA, dict(dO=dO, Wt=Wt), oracle.bwd_data(dO, Wt, H, W, stride, pad)))
    ran = 0
    for v in VARIANTS:
        monkeypatch.setenv("CONVMI_IGEMM_PATCH", v)
        L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
        try:
            for which, code, kw, ref in cases:
                if conv.conv_describe(L.h, code).startswith("igemm_patch "):  # (a patch that fits)
                    ran += 1
                    assert_close(run_pass(L, which, **kw), ref, conv.CONV_BF16, "%s %s" % (which, v))
        finally:
            L.close()
    assert ran >= 4


def test_patch_kernel_fused_operators(monkeypatch):
    """Scale, bias, residual (the output buffer itself) and ReLU, as on the other kernels."""
    import torch
    shape = (3, 72, 40, 9, 11, 3, 3, 1, 1)
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, _ = make_inputs(shape, conv.CONV_BF16, layer_id=9)
    rng = np.random.default_rng(5)
    scale, bias = (rng.uniform(-1, 1, K).astype(np.float32) for _ in range(2))
    from paper_1808_05567_amd import inputs
    resid = inputs.round_to_bf16(rng.uniform(-1, 1, (N, K, H, W)).astype(np.float32))
    ref = oracle.fwd(I, Wt, stride, pad) * scale[None, :, None, None] + bias[None, :, None, None] + resid
    ref = np.maximum(ref, 0)
    for v in VARIANTS:
        monkeypatch.setenv("CONVMI_IGEMM_PATCH", v)
        L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
        try:
            assert conv.conv_describe(L.h, conv.PASS_FWD).startswith("igemm_patch ")
            L.set_input(I)
            L.set_weights(Wt)
            conv.conv_pack_out(L.h, torch.from_numpy(resid).to("cuda", torch.bfloat16), L.out_blk)
            pc = [torch.zeros(L.info.Kp, device="cuda") for _ in range(2)]
            pc[0][:K], pc[1][:K] = torch.from_numpy(scale).cuda(), torch.from_numpy(bias).cuda()
            L.fwd_fused(bias=pc[1], residual=L.out_blk, relu=True, scale=pc[0])
            assert_close(L.get_output().float().cpu().numpy(), ref, conv.CONV_BF16, v)
        finally:
            L.close()


def test_patch_kernel_keeps_images_apart(monkeypatch):
    """A patch holds pixels of the neighbouring image: what is infinite or NaN there stays there."""
    shape = (3, 40, 40, 5, 6, 3, 3, 1, 1)
    I, Wt, _ = make_inputs(shape, conv.CONV_BF16, layer_id=9)
    ref = oracle.fwd(I, Wt, 1, 1)
    I[1] = np.nan
    I[1, :, ::2] = np.inf
    for v in VARIANTS:
        monkeypatch.setenv("CONVMI_IGEMM_PATCH", v)
        L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
        try:
            got = run_pass(L, "fwd", I=I, Wt=Wt)
        finally:
            L.close()
        for n in (0, 2):
            assert_close(got[n], ref[n], conv.CONV_BF16, "image %d, variant %s" % (n, v))
        assert np.isnan(got[1]).all()


@pytest.mark.parametrize("shape", [(4, 3, 64, 30, 31, 5, 5, 2, 2),      # classes as the rows of one 3x3 filter
                                   (3, 8, 40, 18, 20, 5, 5, 2, 2),
                                   (2, 24, 40, 22, 23, 7, 7, 3, 3)],    # a launch per class, most of them 2x2 and 3x3 taps
                         ids=lambda s: "x".join(map(str, s)))
def test_residue_classes_of_strided_backward_passes(shape, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, conv.CONV_BF16, layer_id=9)
    ref = oracle.bwd_data(dO, Wt, H, W, stride, pad)
    ran = 0
    for v in VARIANTS:
        monkeypatch.setenv("CONVMI_IGEMM_PATCH", v)
        L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
        try:
            text = conv.conv_describe(L.h, conv.PASS_BWD_DATA)
            if text.startswith("igemm_patch "):
                assert "forward_weights=1" not in text
                ran += 1
                assert_close(run_pass(L, "bwd", Wt=Wt, dO=dO), ref, conv.CONV_BF16, v)
        finally:
            L.close()
    assert ran >= 2
