"""bf16 3x3 layers of few channels with the weights in registers (igemm_stream.hip), forward and backward, against the oracle: ragged
channel counts, image ends inside a step, rows wider and narrower than a chunk of the ring, one step and many."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

BF16 = conv.CONV_BF16
SHAPES = [(2, 64, 64, 56, 56), (3, 32, 64, 9, 11), (5, 48, 40, 7, 7), (1, 64, 96, 12, 147), (2, 24, 136, 17, 63), (2, 36, 20, 13, 64), (1, 8, 8, 3, 2),
          (40, 64, 48, 20, 20), (1, 60, 60, 70, 127), (300, 32, 32, 13, 14)]
IDS = dict(ids=lambda s: "x".join(map(str, s)))


def _layer(shape, env):
    with pytest.MonkeyPatch.context() as mp:
        mp.setenv("CONVMI_STREAM", env)
        return conv.ConvLayer(*shape, 3, 3, 1, 1, dtype=BF16)


@pytest.mark.parametrize("rows", ["1", "2"])
@pytest.mark.parametrize("shape", SHAPES, **IDS)
def test_matches_oracle(shape, rows):
    N, C, K, H, W = shape
    full = shape + (3, 3, 1, 1)
    I, Wt, dO = make_inputs(full, BF16, layer_id=71)
    L = _layer(shape, rows)
    try:
        ran = 0
        for which, pass_, red in (("fwd", conv.PASS_FWD, C), ("bwd", conv.PASS_BWD_DATA, K)):
            on = " instead=igemm_stream," in conv.conv_describe(L.h, pass_)
            assert on or red > 64 or W > 127, (which, conv.conv_describe(L.h, pass_))
            if not on:
                continue
            ran += 1
            ref = oracle.fwd(I, Wt, 1, 1) if which == "fwd" else oracle.bwd_data(dO, Wt, H, W, 1, 1)
            kw = dict(I=I, Wt=Wt) if which == "fwd" else dict(dO=dO, Wt=Wt)
            print(shape, which, rows, flush=True)
            assert_close(run_pass(L, which, **kw), ref, BF16, which)
        assert ran or W > 127
    finally:
        L.close()


# The widest rows of three and of four chunks of the ring, and one more: more than eight steps a workgroup, so that the ring comes round.
# Layer, then groups of 32 result channels that fit the LDS forward and backward.
WIDE = [((3, 64, 32, 430, 255), "1", "12"), ((2, 40, 64, 700, 192), "12", "1"), ((2, 32, 40, 690, 191), "12", "12"), ((2, 32, 40, 690, 256), "", "")]


@pytest.mark.parametrize("rows", ["1", "2"])
@pytest.mark.parametrize("shape,fwd,bwd", WIDE, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else s or "none")
def test_rows_that_leave_the_ring_no_slack(shape, fwd, bwd, rows):
    N, C, K, H, W = shape
    I, Wt, dO = make_inputs(shape + (3, 3, 1, 1), BF16, layer_id=74)
    L = _layer(shape, rows)
    try:
        for which, pass_, fits in (("fwd", conv.PASS_FWD, fwd), ("bwd", conv.PASS_BWD_DATA, bwd)):
            on = conv.conv_describe(L.h, pass_).partition(" instead=igemm_stream,")[2]
            assert bool(on) == (rows in fits), (which, on)
            if not on:
                continue
            assert int(on.partition("steps")[2].partition(",")[0]) > 8, on
            print(shape, which, rows, flush=True)
            ref = oracle.fwd(I, Wt, 1, 1) if which == "fwd" else oracle.bwd_data(dO, Wt, H, W, 1, 1)
            assert_close(run_pass(L, which, **(dict(I=I, Wt=Wt) if which == "fwd" else dict(dO=dO, Wt=Wt))), ref, BF16, which)
    finally:
        L.close()


def test_infinities_reach_the_pixels_around_them_only():
    shape = (2, 40, 64, 11, 13)
    I, Wt, _ = make_inputs(shape + (3, 3, 1, 1), BF16, layer_id=72)
    I[0, 3, 0, 12] = np.inf
    I[0, 39, 10, 0] = np.nan
    I[1, 5, 5, 5] = -np.inf
    with np.errstate(invalid="ignore"):
        ref = oracle.fwd(I, Wt, 1, 1)
    fine = np.isfinite(ref)
    L = _layer(shape, "2")
    try:
        got = run_pass(L, "fwd", I=I, Wt=Wt).astype(np.float64)
    finally:
        L.close()
    assert np.array_equal(np.isfinite(got), fine)
    assert np.array_equal(got[~fine], ref[~fine], equal_nan=True)
    assert_close(np.where(fine, got, 0), np.where(fine, ref, 0), BF16)


@pytest.mark.parametrize("shape,fwd,bwd", [((16, 32, 64, 147, 147), True, True), ((256, 64, 64, 56, 56), False, False), ((8, 64, 64, 56, 56), False, False),
                                           ((222, 32, 24, 28, 31), False, True)],
                         ids=lambda s: str(s) if isinstance(s, bool) else "x".join(map(str, s)))
def test_chosen_and_the_same_as_the_staged_kernel(shape, fwd, bwd):
    """Which kernel runs on either side of the line, and all its results against the other kernel's: the sums differ in their order, so
    a result is the same or the next bf16 number (2^-7 of it)."""
    N, C, K, H, W = shape
    got = {}
    for env in ("any", "0"):
        L = conv.ConvLayer(*shape, 3, 3, 1, 1, dtype=BF16) if env == "any" else _layer(shape, env)
        try:
            on = [" instead=igemm_stream," in conv.conv_describe(L.h, p) for p in (conv.PASS_FWD, conv.PASS_BWD_DATA)]
            assert on == ([fwd, bwd] if env == "any" else [False, False])
            if not (fwd or bwd):
                return
            I, Wt, dO = make_inputs(shape + (3, 3, 1, 1), BF16, layer_id=73)
            got[env] = (run_pass(L, "fwd", I=I, Wt=Wt), run_pass(L, "bwd", dO=dO, Wt=Wt))
        finally:
            L.close()
    for a, b in zip(got["any"], got["0"]):
        rms = np.sqrt(np.mean(np.square(b, dtype=np.float64)))
        assert (np.abs(a - b) <= 2.0 ** -7 * np.abs(b) + 1e-5 * rms).all()
        assert np.count_nonzero(a != b) <= 1e-3 * a.size  # (a sum's error is 1e-7 of it: few lie that close to the middle)
