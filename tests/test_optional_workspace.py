"""A backward pass or update that only the untiled kernels served took no workspace.  With a tiled kernel for
it, a caller that brings none, or too little of one, must still be served (by the untiled kernel)."""
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs

BWD = [(2, 20, 24, 9, 11, 1, 5, 1, (0, 2)), (3, 24, 36, 9, 9, 3, 3, 2, 1)]


@pytest.mark.parametrize("shape", BWD, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_checked_entry_point_accepts_no_workspace(shape):
    """Host only: the misaligned dI is what stops the calls, after the size check."""
    lib = conv.load()
    h = conv.conv_create(*shape, 0)
    try:
        assert conv.conv_describe(h, conv.PASS_BWD_DATA).startswith("igemm")
        assert conv.conv_query(h).workspace_bytes > 16
        assert lib.conv_bwd_data_ws(h, 16, 16, 8, None, 0, None) == conv.CONV_EINVAL
        assert lib.conv_bwd_data_ws(h, 16, 16, 8, 16, 16, None) == conv.CONV_EINVAL
    finally:
        conv.conv_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", BWD + [(2, 64, 32, 12, 12, 7, 7, 1, 3)], ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_backward_with_and_without_a_workspace(shape, dtype):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, dtype, layer_id=14)
    ref = oracle.bwd_data(dO, Wt, H, W, stride, pad)
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        L.set_outgrad(dO)
        L.set_weights(Wt)
        for ws in (L.ws, None):
            L.ws.fill_(0xFF)
            L.in_blk.fill_(float("nan"))
            conv.conv_bwd_data(L.h, L.out_blk, L.wt_blk, L.in_blk, ws)
            assert_close(L.get_input().float().cpu().numpy(), ref, dtype, "bwd, workspace %s" % (ws is not None))
        L.in_blk.fill_(float("nan"))
        conv.conv_bwd_data_noalloc(L.h, L.out_blk, L.wt_blk, L.in_blk)
        assert_close(L.get_input().float().cpu().numpy(), ref, dtype, "bwd, static scratch")
    finally:
        L.close()
