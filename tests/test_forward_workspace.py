"""The forward pass needs a workspace only where its plan splits the reduction over workgroups: elsewhere NULL is
as good as a buffer, also for results of few tiles, and the size-checked entry point asks for nothing."""
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs

DTYPES = [pytest.param(conv.CONV_F32, id="f32"), pytest.param(conv.CONV_BF16, id="bf16")]
SHAPES = [(1, 256, 256, 14, 14, 3, 3, 1, 1), (1, 512, 96, 7, 7, 3, 3, 1, 1), (2, 64, 40, 9, 9, 1, 1, 1, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward_takes_no_workspace_that_it_does_not_use(shape, dtype, monkeypatch):
    lib = conv.load()
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, _ = make_inputs(shape, dtype, layer_id=3)
    ref = oracle.fwd(I, Wt, stride, pad)
    for v in ("1,1,8,1", "1,1,8,2"):  # one split, several
        monkeypatch.setenv("CONVMI_IGEMM_REG", v)
        L = conv.ConvLayer(*shape, dtype=dtype)
        try:
            split = " ksplit=1 " not in conv.conv_describe(L.h, conv.PASS_FWD)
            L.set_input(I)
            L.set_weights(Wt)
            ptr = [t.data_ptr() for t in (L.in_blk, L.wt_blk, L.out_blk)]
            if split:
                assert lib.conv_fwd(L.h, *ptr, None, None) == conv.CONV_EWORKSPACE
                assert lib.conv_fwd_ws(L.h, *ptr, L.ws.data_ptr(), 0, None) == conv.CONV_EWORKSPACE
                continue
            for entry in (lambda: conv.conv_fwd(L.h, L.in_blk, L.wt_blk, L.out_blk, None),
                          lambda: conv.conv_fwd_ws(L.h, L.in_blk, L.wt_blk, L.out_blk, None)):
                L.out_blk.fill_(float("nan"))
                entry()
                assert_close(L.get_output().float().cpu().numpy(), ref, dtype, "forward without a workspace")
        finally:
            L.close()
