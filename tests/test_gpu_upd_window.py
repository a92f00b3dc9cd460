"""Weight update of strided bf16 layers with one window of the input for all taps of a filter row, with one split (dW
written directly) and several, against the oracle at the edges: rows shorter than a quad of pixels, than a stage and
than a tap's reach, runs that end inside a stage, rows whose window reaches past their last pixel, ragged channels
both ways, more padding than "same".  Bars: gpu_util.assert_close for an fp32 result."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

VARIANT = "2,2,8,3"

# N, C, K, H, W, R, S, stride, pad
SHAPES = [
    (1, 20, 24, 3, 3, 3, 3, 2, 1),          # every row shorter than a quad
    (1, 12, 20, 4, 1, 1, 3, 2, (0, 1)),     # ... a single column
    (5, 64, 64, 14, 14, 3, 3, 2, 1),        # even extents: no dead slot, the last column is the last tap's
    (9, 72, 136, 7, 7, 3, 3, 2, 1),         # several rows to a stage; ragged channels
    (2, 40, 100, 13, 15, 3, 3, 2, 1),       # odd extents
    (3, 36, 32, 11, 9, 3, 3, 2, 0),         # no padding: a slot more than pixels to a row
    (3, 33, 65, 10, 34, 3, 3, 2, 0),        # ... even extents: one column is never read
    (1, 12, 40, 5, 150, 3, 3, 2, 1),
    (2, 16, 24, 9, 7, 2, 3, 2, (1, 2)),     # an even number of filter rows, more padding than "same"
    (1, 16, 24, 9, 9, 3, 3, 2, (1, 4)),     # the most padding it takes
]


def ids(s):
    return "x".join(map(str, s)).replace(" ", "")


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_window_update_matches_oracle(shape, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, conv.CONV_BF16, layer_id=12)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    for splits in (1, 3):
        monkeypatch.setenv("CONVMI_UPD_WINDOW", "%s,%d" % (VARIANT, splits))
        L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
        try:
            d = conv.conv_describe(L.h, conv.PASS_UPD)
            assert d.startswith("upd_ring ") and "window=" in d and "window=0" not in d
            got = run_pass(L, "upd", I=I, dO=dO)
            assert np.isfinite(L.dwt_blk.cpu().numpy()).all()  # (padded channel slots too)
        finally:
            L.close()
        assert_close(got, ref, conv.CONV_F32, "splits %d" % splits)


@pytest.mark.parametrize("shape", [(3, 32, 32, 7, 7, 3, 3, 2, 1), (2, 32, 32, 10, 12, 3, 3, 2, 1),
                                   (2, 32, 32, 11, 13, 3, 3, 2, 0), (2, 32, 32, 6, 8, 3, 3, 2, 0)], ids=ids)
def test_what_a_tap_does_not_read_does_not_reach_it(shape, monkeypatch):
    """Infinite inputs in the first and the last column: dW is infinite or NaN exactly where a tap reads them."""
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, conv.CONV_BF16, layer_id=12)
    I[0, 3, :, 0] = np.inf
    I[0, 5, :, W - 1] = np.inf
    ref = oracle.upd(I, dO, R, S, stride, pad)
    monkeypatch.setenv("CONVMI_UPD_WINDOW", "%s,2" % VARIANT)
    L = conv.ConvLayer(*shape, dtype=conv.CONV_BF16)
    try:
        got = run_pass(L, "upd", I=I, dO=dO)
    finally:
        L.close()
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    ok = np.isfinite(ref)
    assert_close(np.where(ok, got, 0.0), np.where(ok, ref, 0.0), conv.CONV_F32)
