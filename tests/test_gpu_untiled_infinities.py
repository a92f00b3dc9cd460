"""Layers without a staged kernel, whose forward and backward passes run on the register-operand kernel in the place
of the untiled loops: as on those, a tap outside the image contributes nothing, also where the weight that it would
meet is infinite or NaN, and a residue class without taps is zero whatever dO holds.  Against the oracle, which
walks the same taps: the same infinities and NaNs in the same places, gpu_util.assert_close elsewhere."""
import numpy as np
import pytest

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

DTYPES = [pytest.param(conv.CONV_F32, id="f32"), pytest.param(conv.CONV_BF16, id="bf16")]

# N, C, K, H, W, R, S, stride, pad
BWD = [
    (2, 20, 24, 9, 11, 1, 5, 1, (0, 2)),
    (3, 24, 36, 9, 9, 3, 3, 2, 1),            # odd blocks of channels: four residue classes
    (2, 16, 24, 9, 10, 1, 9, 2, (0, 4)),      # classes without taps
    (2, 12, 20, 8, 9, 2, 4, 3, (1, 2)),       # nine classes
    (2, 64, 32, 12, 12, 7, 7, 1, 3),
]
FWD = [(8, 64, 64, 24, 24, 1, 5, 1, (0, 2)), (20, 40, 72, 25, 21, 2, 5, 2, (1, 2)), (6, 48, 64, 21, 20, 6, 6, 1, 3)]


def _spoil(t, rng):
    """A few infinities and a NaN, so that most results stay finite."""
    flat = t.reshape(-1)
    flat[rng.choice(flat.size, 3, replace=False)] = [np.inf, -np.inf, np.nan]


def _assert_same(got, ref, dtype, what):
    got = np.asarray(got, np.float64)
    fine = np.isfinite(ref)
    wrong = int((fine != np.isfinite(got)).sum())
    assert wrong == 0, (what, wrong)
    same = np.array_equal(got[~fine], ref[~fine], equal_nan=True)
    assert same, what
    assert fine.mean() > 0.2 and not fine.all(), (what, float(fine.mean()))
    assert_close(np.where(fine, got, 0), np.where(fine, ref, 0), dtype, what)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", BWD, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_backward_leaves_out_taps_outside_the_image(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, dtype, layer_id=21)
    rng = np.random.default_rng(3)
    for spoiled in (Wt, dO):
        keep = spoiled.copy()
        _spoil(spoiled, rng)
        ref = oracle.bwd_data(dO, Wt, H, W, stride, pad)
        for v in (None, "1,1,8,3", "2,2,4"):
            if v:
                monkeypatch.setenv("CONVMI_IGEMM_REG", v)
            L = conv.ConvLayer(*shape, dtype=dtype)
            monkeypatch.delenv("CONVMI_IGEMM_REG", raising=False)
            try:
                assert conv.conv_describe(L.h, conv.PASS_BWD_DATA).startswith("igemm_reg ")
                _assert_same(run_pass(L, "bwd", Wt=Wt, dO=dO), ref, dtype, "bwd, variant %s" % v)
            finally:
                L.close()
        spoiled[...] = keep


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", FWD, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_forward_leaves_out_taps_outside_the_image(shape, dtype):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, _ = make_inputs(shape, dtype, layer_id=22)
    _spoil(Wt, np.random.default_rng(4))
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        assert conv.conv_describe(L.h, conv.PASS_FWD).startswith("igemm_reg ")
        _assert_same(run_pass(L, "fwd", I=I, Wt=Wt), oracle.fwd(I, Wt, stride, pad), dtype, "fwd")
    finally:
        L.close()


@pytest.mark.parametrize("shape", [(2, 6661, 16764, 8, 10, 3, 3, 2, 0), (2, 6228, 12075, 74, 74, 3, 3, 2, 0)],
                         ids=lambda s: "x".join(map(str, s)))
def test_update_left_to_the_untiled_loop_stays_there(shape):
    """Partial copies that dwarf the tensors: no tiled update (host only)."""
    h = conv.conv_create(*shape)
    try:
        assert conv.conv_describe(h, conv.PASS_UPD).startswith("direct ")
    finally:
        conv.conv_destroy(h)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", BWD, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_all_residue_classes_run_on_the_same_kind_of_kernel(shape, dtype):
    """A pass in which one class has a staged kernel and another has not (host only; (2, 16, 24) above: the class
    without taps is a 1x1 filter).  The description is the first class's."""
    h = conv.conv_create(*shape, dtype)
    try:
        assert conv.conv_describe(h, conv.PASS_BWD_DATA).startswith("igemm_reg ")
    finally:
        conv.conv_destroy(h)
