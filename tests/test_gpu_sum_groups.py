"""fp32 sums in groups: a wave's part of a reduction (forward, register-operand and 64 x 128 staged kernels) and its
pixels of a weight update (ring kernel) are summed in groups from zero where one chain would have the larger rounding
error.  Against the oracle at the groups' edges, and the error itself against 64 bits for layers whose reduction
used to be split over more chains.  Bars: gpu_util.assert_close, and see PRECISION."""
import numpy as np
import pytest
import torch

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, run_pass

pytestmark = pytest.mark.gpu

F32, BF16 = conv.CONV_F32, conv.CONV_BF16

REG = ["1,1,4", "1,1,8", "2,1,8", "1,2,4", "2,2,4", "1,1,8,2"]
REG_SHAPES = [(2, 72, 40, 9, 7, 3, 3, 1, 1), (1, 520, 36, 7, 7, 1, 1, 1, 0), (1, 8, 32, 5, 5, 1, 1, 1, 0)]


@pytest.mark.parametrize("group", [1, 2, 5])
@pytest.mark.parametrize("shape", REG_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_register_operand_kernel(shape, group, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, _ = make_inputs(shape, F32, layer_id=31)
    ref = oracle.fwd(I, Wt, stride, pad)
    monkeypatch.setenv("CONVMI_IGEMM_GROUP", str(group))
    for v in REG:
        monkeypatch.setenv("CONVMI_IGEMM_REG", v)
        L = conv.ConvLayer(*shape, dtype=F32)
        try:
            text = conv.conv_describe(L.h, conv.PASS_FWD)
            assert text.startswith("igemm_reg ") and " group=%d " % group in text
            assert_close(run_pass(L, "fwd", I=I, Wt=Wt), ref, F32, "variant %s" % v)
        finally:
            L.close()


@pytest.mark.parametrize("group", [1, 2, 3, 9])
@pytest.mark.parametrize("shape", [(3, 64, 136, 13, 15, 3, 3, 1, 1), (3, 64, 80, 12, 13, 1, 1, 1, 0), (2, 8, 80, 9, 9, 3, 3, 1, 1),
                                   (2, 96, 64, 17, 17, 1, 7, 1, (0, 3))], ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_staged_kernel(shape, group, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, _ = make_inputs(shape, F32, layer_id=32)
    ref = oracle.fwd(I, Wt, stride, pad)
    monkeypatch.setenv("CONVMI_IGEMM_GROUP", str(group))
    monkeypatch.setenv("CONVMI_IGEMM_CAND", "2,2,1,2,2,%d" % (4 if R * S == 1 else 2))
    L = conv.ConvLayer(*shape, dtype=F32)
    try:
        text = conv.conv_describe(L.h, conv.PASS_FWD)
        assert " waves=2x2 frags=1x2 " in text and " group=%d " % group in text
        assert_close(run_pass(L, "fwd", I=I, Wt=Wt), ref, F32, "group %d" % group)
    finally:
        L.close()


# columns, type: variants with their summations apart (1: groups, 2: by the stage)
RING = {(1, F32): ["1,1,8,4,%d,1", "2,2,8,2,%d,1"], (3, F32): ["1,1,8,2,%d,1", "1,2,8,2,%d,1", "2,2,8,2,%d,2", "2,2,4,4,%d,2"],
        (5, F32): ["1,1,8,2,%d,1"], (7, F32): ["1,1,8,2,%d,2"], (1, BF16): ["1,1,8,4,%d,1", "2,2,8,2,%d,1"],
        (3, BF16): ["1,1,8,2,%d,1", "1,2,8,2,%d,1"], (5, BF16): ["1,1,8,2,%d,1"]}
RING_SHAPES = [(1, 32, 32, 1, 1, 1, 1, 1, 0), (3, 72, 136, 17, 15, 1, 1, 1, 0), (3, 64, 64, 14, 14, 3, 3, 1, 1), (2, 40, 100, 27, 31, 3, 3, 2, 1),
               (2, 40, 36, 19, 21, 5, 5, 1, 2), (2, 40, 48, 17, 17, 1, 7, 1, (0, 3))]


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", RING_SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_ring_update(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, dtype, layer_id=33)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    for v in RING.get((S, dtype), []):
        for splits in (1, 2):
            for group in ((1, 2, 3) if v.endswith("1") else (0,)):
                monkeypatch.setenv("CONVMI_UPD_RING", (v % splits) + (",%d" % group if group else ""))
                L = conv.ConvLayer(*shape, dtype=dtype)
                try:
                    assert " sum=%s group=%d " % (v[-1], group) in conv.conv_describe(L.h, conv.PASS_UPD)
                    got = run_pass(L, "upd", I=I, dO=dO)
                    assert np.isfinite(L.dwt_blk.cpu().numpy()).all()
                finally:
                    L.close()
                assert_close(got, ref, F32, "%s splits %d group %d" % (v, splits, group))


# Layer, pass, type, largest relative error (2-norm) against 64 bits.  The bound is 1.15 times the error of the
# kernels that these layers ran on when their reduction was split over more workgroups, waves and copies (the
# spread between inputs is under 2 %); in one chain per wave they had 1.5 to 2.8 times that error.
PRECISION = [
    ((64, 512, 512, 7, 7, 3, 3, 1, 1), "fwd", F32, 4.04e-7),
    ((28, 448, 384, 8, 8, 3, 3, 1, 1), "fwd", F32, 2.60e-7),
    ((8, 512, 1024, 28, 28, 1, 1, 2, 0), "fwd", F32, 1.55e-7),
    ((8, 2048, 512, 7, 7, 1, 1, 1, 0), "fwd", F32, 1.80e-7),
    ((64, 192, 320, 17, 17, 3, 3, 2, 0), "upd", F32, 1.91e-7),
    ((28, 128, 128, 28, 28, 3, 3, 1, 1), "upd", F32, 2.61e-7),
    ((8, 256, 1024, 14, 14, 1, 1, 1, 0), "upd", F32, 1.28e-7),
    ((64, 48, 64, 35, 35, 5, 5, 1, 2), "upd", F32, 2.58e-7),
    ((28, 256, 256, 14, 14, 3, 3, 1, 1), "upd", BF16, 9.54e-8),
    ((64, 1280, 448, 8, 8, 1, 1, 1, 0), "upd", BF16, 8.95e-8),
]


def _exact(which, a, b, R, S, stride, pad, P, Q):
    """The pass in 64 bits, a matrix product per filter tap: a is the input; b the weights (fwd) or dO (upd)."""
    N, C = a.shape[:2]
    x = torch.nn.functional.pad(a, (pad, pad, pad, pad))
    taps = lambda r, s: x[:, :, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride]  # noqa: E731
    if which == "fwd":
        y = torch.zeros((b.shape[0], N * P * Q), dtype=torch.float64, device=a.device)
        for r in range(R):
            for s in range(S):
                y.addmm_(b[:, :, r, s].contiguous(), taps(r, s).permute(1, 0, 2, 3).reshape(C, N * P * Q))
        return y.reshape(-1, N, P, Q).permute(1, 0, 2, 3)
    K = b.shape[1]
    g = b.permute(1, 0, 2, 3).reshape(K, N * P * Q)
    dw = torch.zeros((K, C, R, S), dtype=torch.float64, device=a.device)
    for r in range(R):
        for s in range(S):
            dw[:, :, r, s] = torch.mm(g, taps(r, s).permute(0, 2, 3, 1).reshape(N * P * Q, C))
    return dw


@pytest.mark.parametrize("shape,which,dtype,before", PRECISION,
                         ids=["%s-%s-%s" % (w, "x".join(map(str, s)), "bf16" if d else "f32") for s, w, d, _ in PRECISION])
def test_error_against_64_bits_is_no_larger_than_that_of_more_chains(shape, which, dtype, before):
    N, C, K, H, W, R, S, stride, pad = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    t = torch.float32 if dtype == F32 else torch.bfloat16
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    x = torch.rand((N, C, H, W), generator=g, device="cuda").mul_(2).sub_(1).to(t)
    b = (torch.randn((K, C, R, S), generator=g, device="cuda").mul_((2.0 / (C * R * S)) ** 0.5) if which == "fwd"
         else torch.rand((N, K, P, Q), generator=g, device="cuda").mul_(2).sub_(1)).to(t)
    ref = _exact(which, x.double(), b.double(), R, S, stride, pad, P, Q)
    L = conv.ConvLayer(*shape, dtype=dtype)
    try:
        conv.conv_pack_in(L.h, x, L.in_blk)
        if which == "fwd":
            conv.conv_pack_wt(L.h, b, L.wt_blk)
            L.fwd()
            got = L.get_output()
        else:
            conv.conv_pack_out(L.h, b, L.out_blk)
            L.upd()
            got = L.get_dweights()
        err = float((got.double() - ref).norm() / ref.norm())
    finally:
        L.close()
    assert err <= 1.15 * before, (err, before)
