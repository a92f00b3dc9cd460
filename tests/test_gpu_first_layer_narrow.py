"""Weight update of first layers (at most four input channels) with at most 32 output channels, which give all eight
waves to the pixels, and with just over 32, against the oracle: every number of accumulator tiles, rows shorter than the waves'
pairs and not a multiple of them, bands that cross images.  Bars: gpu_util.assert_close for an fp32 result."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 3, 32, 5, 5, 3, 3, 2, 0),       # two pixels a row
    (3, 3, 32, 11, 13, 3, 3, 2, 0),
    (2, 3, 20, 30, 75, 3, 3, 2, 0),     # 37 columns: pairs past the row's end
    (2, 1, 8, 9, 67, 3, 3, 1, 1),
    (2, 4, 32, 20, 21, 3, 3, 2, 1),     # two tiles
    (1, 1, 32, 15, 14, 7, 7, 2, 3),
    (2, 2, 12, 17, 18, 7, 7, 2, 3),
    (2, 3, 32, 24, 25, 7, 7, 2, 3),
    (1, 4, 32, 13, 40, 7, 7, 1, 3),
    (2, 3, 36, 30, 75, 3, 3, 2, 0),     # two waves along the channels
]


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_narrow_first_layer_update_matches_oracle(shape, dtype):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, dtype, layer_id=1)
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert conv.conv_describe(L.h, conv.PASS_UPD).startswith("upd_c4")
        got = run_pass(L, "upd", I=I, dO=dO)
        assert np.isfinite(L.dwt_blk.cpu().numpy()).all()  # (the slots without a channel too)
    finally:
        L.close()
    assert_close(got, oracle.upd(I, dO, R, S, stride, pad), conv.CONV_F32, "update")
