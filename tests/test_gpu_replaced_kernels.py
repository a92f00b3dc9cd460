"""Kernels that others have taken over from at most sizes, where those are kept out by their tuning variables: the band, row,
flat and general update kernels (strips of columns, launches per filter row, partial copies of every number) and the
untiled forward and backward loops.  Against the oracle; bars: gpu_util.assert_close."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

F32, BF16 = conv.CONV_F32, conv.CONV_BF16

# N, C, K, H, W, R, S, stride, pad; kernel in fp32, in bf16
UPD = [
    ((3, 300, 72, 9, 11, 1, 1, 1, 0), "upd_1x1", "upd_1x1"),
    ((2, 48, 264, 12, 9, 1, 1, 2, 0), "upd_1x1", "upd_1x1"),
    ((5, 64, 40, 13, 15, 1, 1, 1, 0), "upd ", "upd_1x1"),
    ((5, 64, 96, 14, 14, 3, 3, 1, 1), "upd_bands", "upd_rows"),
    ((2, 72, 136, 27, 19, 3, 3, 1, 1), "upd_bands", "upd_rows"),
    ((2, 40, 72, 13, 15, 3, 3, 2, 1), "upd ", "upd_rows"),
    ((2, 32, 64, 20, 147, 3, 3, 1, 1), "upd_bands", "upd_rows"),       # strips of columns
    ((4, 64, 64, 17, 17, 7, 1, 1, (3, 0)), "upd ", "upd_rows"),
    ((4, 64, 72, 17, 17, 1, 7, 1, (0, 3)), "upd_bands", "upd_rows"),
    ((4, 48, 64, 35, 35, 5, 5, 1, 2), "upd ", "upd_rows"),                # a launch per filter row
]


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", UPD, ids=lambda c: "x".join(map(str, c[0])).replace(" ", ""))
def test_update_without_the_ring_kernel(case, dtype, monkeypatch):
    shape, f32, bf16 = case
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, dtype, layer_id=51)
    monkeypatch.setenv("CONVMI_UPD_RING", "0")
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert conv.conv_describe(L.h, conv.PASS_UPD).startswith(f32 if dtype == F32 else bf16)
        got = run_pass(L, "upd", I=I, dO=dO)
        assert np.array_equal(got, run_pass(L, "upd", I=I, dO=dO))
    finally:
        L.close()
    assert_close(got, oracle.upd(I, dO, R, S, stride, pad), F32, "update")


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
def test_untiled_forward_with_fused_operators(dtype, monkeypatch):
    import torch
    shape = (2, 20, 24, 9, 11, 1, 5, 1, (0, 2))
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, res = make_inputs(shape, dtype, layer_id=52)
    rng = np.random.default_rng(6)
    scale, bias = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.normal(0, 0.2, K).astype(np.float32)
    ref = oracle.fwd_fused(I, Wt, stride, pad, bias=bias, residual=res, relu=True, scale=scale)
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert conv.conv_describe(L.h, conv.PASS_FWD).startswith("direct ")
        assert conv.conv_describe(L.h, conv.PASS_BWD_DATA).startswith("direct ")
        L.set_input(I)
        L.set_weights(Wt)
        L.set_outgrad(res)
        pc = []
        for a in (scale, bias):
            t = torch.zeros(L.info.Kp, dtype=torch.float32, device=L.device)
            t[:K] = torch.from_numpy(a)
            pc.append(t)
        L.fwd_fused(bias=pc[1], residual=L.out_blk, relu=True, scale=pc[0])
        assert_close(L.get_output().float().cpu().numpy(), ref, dtype, "fused")
    finally:
        L.close()
