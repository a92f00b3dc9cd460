"""Backward by data reading the forward pass's weights in the staged kernel (every tile it is built in), in the residue
classes of a strided pass and in the register-operand kernel, against the oracle at the edges: ragged channels both
ways (an odd number of channel blocks), one pixel, images smaller than a tile, tiles
that cross images, padding other than "same", the scattering store.  The workspace holds NaN patterns: nothing may be
read from it.  Bars: gpu_util.assert_close."""
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

# waves over channels, over pixels, fragments of both, buffers, channel blocks to a step
TILES_1X1 = {conv.CONV_BF16: ["2,2,1,2,2,4", "2,2,2,2,2,4", "2,2,1,2,2,8", "2,2,2,2,2,8", "4,1,1,7,2,4", "4,1,1,7,3,4",
                              "2,2,1,7,2,4", "2,2,1,7,3,4", "4,2,2,4,2,8", "2,2,2,4,2,4", "4,1,1,7,2,8"],
             conv.CONV_F32: ["2,2,1,2,2,4", "2,2,2,2,2,4", "2,2,1,2,2,8", "2,2,2,2,2,8", "4,1,1,7,2,4", "2,2,1,7,2,4"]}
TILES = {conv.CONV_BF16: ["2,2,1,2,2,2", "2,2,2,2,2,2", "1,4,2,4,2,2", "2,4,2,4,2,2"],
         conv.CONV_F32: ["2,2,1,2,2,2", "2,2,2,2,2,2", "4,1,1,7,2,2", "2,2,1,7,2,2", "1,4,1,7,2,2"]}

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 8, 64, 1, 1, 1, 1, 1, 0),
    (5, 72, 64, 7, 9, 1, 1, 1, 0),            # one step, or two
    (3, 264, 160, 13, 11, 1, 1, 1, 0),        # channels beyond a tile
    (3, 40, 192, 9, 10, 1, 1, 2, 0),          # the scattering store
    (5, 40, 48, 7, 7, 3, 3, 1, 1),
    (2, 136, 32, 13, 15, 3, 3, 1, 0),
    (1, 20, 80, 30, 29, 3, 3, 1, (0, 1)),
    (3, 72, 48, 17, 16, 1, 7, 1, (0, 3)),
    (3, 40, 96, 9, 11, 7, 1, 1, (3, 0)),
]


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_staged_tiles_match_oracle(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, dtype, layer_id=11)
    ref = oracle.bwd_data(dO, Wt, H, W, stride, pad)
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    ran = set()
    for tile in (TILES_1X1 if R * S == 1 else TILES)[dtype]:
        monkeypatch.setenv("CONVMI_IGEMM_CAND", tile)
        L = conv.ConvLayer(*shape, dtype=dtype)
        try:
            text = conv.conv_describe(L.h, conv.PASS_BWD_DATA)
            if "forward_weights=1" in text and "waves=%s frags=%s " % tuple(
                    "x".join(tile.split(",")[i:i + 2]) for i in (0, 2)) in text:
                ran.add(tile)
                L.ws.fill_(0xFF)
                assert_close(run_pass(L, "bwd", Wt=Wt, dO=dO), ref, dtype, tile)
        finally:
            L.close()
    assert len(ran) >= 2, ran


@pytest.mark.parametrize("shape,dtype,env", [
    ((3, 264, 136, 5, 7, 1, 1, 1, 0), conv.CONV_BF16, ("CONVMI_IGEMM_REG", "1,1,8")),
    ((3, 264, 136, 5, 7, 1, 1, 1, 0), conv.CONV_BF16, ("CONVMI_IGEMM_REG", "2,1,8")),
    ((3, 40, 72, 9, 7, 1, 1, 1, 0), conv.CONV_BF16, ("CONVMI_IGEMM_REG", "2,2,4")),
    ((2, 40, 24, 9, 8, 5, 5, 1, 2), conv.CONV_BF16, ("CONVMI_IGEMM_REG", "1,1,4")),
    ((5, 40, 64, 7, 8, 3, 3, 2, 1), conv.CONV_BF16, ("CONVMI_BWD_QUAD", "1")),
    ((5, 36, 48, 7, 8, 3, 3, 2, 0), conv.CONV_F32, ("CONVMI_BWD_QUAD", "1")),
], ids=str)
def test_other_kernels_match_oracle(shape, dtype, env, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, dtype, layer_id=11)
    monkeypatch.setenv(*env)
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert "forward_weights=1" in conv.conv_describe(L.h, conv.PASS_BWD_DATA)
        L.ws.fill_(0xFF)
        assert_close(run_pass(L, "bwd", Wt=Wt, dO=dO), oracle.bwd_data(dO, Wt, H, W, stride, pad), dtype, str(env))
    finally:
        L.close()
