"""fp32 passes on the bf16 matrix instructions (each value as three bf16 numbers): every tile and block size against the oracle at
the edges of its tiles, what is fused into the store, and the values that three bf16 numbers do not hold.  Bars:
gpu_util.assert_close; where the fp32 instructions give an infinity or a NaN, the same one."""
import numpy as np
import pytest
import torch

import oracle
from paper_1808_05567_amd import conv

from gpu_util import assert_close, make_inputs, rel_l2, run_pass

pytestmark = pytest.mark.gpu

F32 = conv.CONV_F32
# "channel waves, pixel waves, fragments, sets, groups of 16 channels, strips" and "r, fragments, waves"
STAGED = ["4,1,4,1", "4,1,2,1", "2,2,4,1", "2,2,2,1", "4,1,4,2", "4,1,2,2", "2,2,4,2", "2,2,2,2"]
IN_REGISTERS = ["r,1,1,4", "r,1,1,8", "r,1,1,16", "r,2,1,4", "r,2,1,8", "r,1,2,4", "r,2,2,4", "r,2,2,8"]
SHAPES = [  # N, C, K, H, W, R, S, stride, pad: ragged channel blocks, images smaller than a tile, wide rows, strides, few taps
    (3, 72, 40, 13, 15, 3, 3, 1, 1), (2, 20, 136, 9, 11, 1, 1, 1, 0), (3, 36, 52, 15, 13, 1, 1, 2, 0), (5, 32, 32, 7, 7, 3, 3, 1, 1),
    (3, 64, 80, 17, 17, 1, 7, 1, (0, 3)), (2, 48, 64, 21, 19, 7, 1, 1, (3, 0)), (3, 64, 64, 15, 17, 3, 3, 2, 1), (2, 36, 24, 15, 17, 3, 3, 2, 0),
    (1, 16, 32, 30, 149, 3, 3, 1, 1), (2, 32, 48, 12, 12, 5, 5, 1, 2), (2, 24, 40, 11, 12, 3, 3, 1, 0), (1, 100, 60, 3, 2, 1, 1, 1, 0),
]
IDS = dict(ids=lambda s: "x".join(map(str, s)).replace(" ", ""))


def _variants(shape, which):
    out = []
    for v in STAGED:
        for g, strips in ((1, 1), (2, 1), (1, 2)):
            out += ["%s,%d,%d,%d" % (v, g, strips, fw) for fw in ((0, 1) if which == "bwd" else (0,))]
    return out + ["%s,%d" % (v, fw) for v in IN_REGISTERS for fw in ((0, 1) if which == "bwd" else (0,))]


def _layer(shape, **env):
    with pytest.MonkeyPatch.context() as mp:
        for k, v in env.items():
            mp.setenv(k, v)
        return conv.ConvLayer(*shape, dtype=F32)


@pytest.mark.parametrize("which", ["fwd", "bwd"])
@pytest.mark.parametrize("shape", SHAPES, **IDS)
def test_forward_and_backward_match_oracle(shape, which):
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, dO = make_inputs(shape, F32, layer_id=51)
    ref = oracle.fwd(I, Wt, stride, pad) if which == "fwd" else oracle.bwd_data(dO, Wt, H, W, stride, pad)
    kw = dict(I=I, Wt=Wt) if which == "fwd" else dict(dO=dO, Wt=Wt)
    seen = set()
    for v in _variants(shape, which):
        L = _layer(shape, CONVMI_IGEMM_SPLIT=v)
        try:
            text = conv.conv_describe(L.h, conv.PASS_FWD if which == "fwd" else conv.PASS_BWD_DATA)
            on = text.partition(" on_bf16x3=")[2]
            if not on or on in seen:  # (the tile does not fit the LDS, or is the same without the last digits)
                continue
            seen.add(on)
            assert_close(run_pass(L, which, **kw), ref, F32, "%s variant %s" % (which, v))
        finally:
            L.close()
    strided_classes = which == "bwd" and R * S > 1 and stride > 1
    assert len(seen) >= (3 if strided_classes else 14 if which == "fwd" else 24), sorted(seen)


UPD = ["1,2,2,2,2,16,16", "1,2,2,4,2,16,16", "1,2,1,2,4,32,32", "1,2,1,2,2,32,32", "1,1,2,2,2,32,32", "1,1,1,2,2,32,32", "1,1,1,2,2,64,64",
       "1,2,1,4,2,16,16", "1,1,1,4,2,32,32", "3,1,1,2,2,32,64", "3,1,1,2,4,32,64", "3,1,1,2,2,16,32", "3,1,1,2,2,16,64", "3,1,1,2,4,16,64",
       "3,1,1,2,4,16,32", "3,1,1,1,4,32,64", "3,1,1,4,2,16,32", "4,1,1,2,2,32,64", "4,1,1,2,4,32,64", "4,1,1,2,2,16,32", "5,1,1,2,2,16,32"]


@pytest.mark.parametrize("shape", SHAPES, **IDS)
def test_update_matches_oracle(shape):
    N, C, K, H, W, R, S, stride, pad = shape
    I, _, dO = make_inputs(shape, F32, layer_id=52)
    ref = oracle.upd(I, dO, R, S, stride, pad)
    ran = 0
    for v in UPD:
        for splits in (1, 3):
            L = _layer(shape, CONVMI_UPD_SPLIT="%s,%d" % (v, splits))
            try:
                if " on_bf16x3=upd_split," not in conv.conv_describe(L.h, conv.PASS_UPD):
                    assert not v.startswith("1,"), v  # (one tap fits everywhere)
                    continue
                ran += 1
                assert_close(run_pass(L, "upd", I=I, dO=dO), ref, F32, "%s splits %d" % (v, splits))
                assert np.isfinite(L.dwt_blk.cpu().numpy()).all()
            finally:
                L.close()
    assert ran >= 18, ran


@pytest.mark.parametrize("variant", ["4,1,4,1,1", "2,2,2,2,1", "r,2,1,8"])
def test_fused_operators(variant):
    """Scale, bias, residual (the output buffer itself) and ReLU."""
    shape = (2, 72, 40, 7, 5, 3, 3, 1, 1)
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, res = make_inputs(shape, F32, layer_id=53)
    rng = np.random.default_rng(5)
    scale, bias = rng.uniform(0.5, 1.5, K).astype(np.float32), rng.normal(0, 0.2, K).astype(np.float32)
    ref = np.maximum(oracle.fwd(I, Wt, stride, pad).astype(np.float64) * scale[:, None, None] + bias[:, None, None] + res, 0)
    L = _layer(shape, CONVMI_IGEMM_SPLIT=variant)
    try:
        assert " on_bf16x3=" in conv.conv_describe(L.h, conv.PASS_FWD)
        L.set_input(I)
        L.set_weights(Wt)
        L.set_outgrad(res)  # (the residual sits in the output buffer)
        per_channel = [torch.nn.functional.pad(torch.from_numpy(a), (0, L.info.Kp - K)).to(L.device) for a in (scale, bias)]
        L.fwd_fused(bias=per_channel[1], residual=L.out_blk, relu=True, scale=per_channel[0])
        assert_close(L.get_output().cpu().numpy(), ref, F32, variant)
    finally:
        L.close()


# which pass, fp32 variant's switch, variants
SPECIAL = [("fwd", "CONVMI_IGEMM_SPLIT", ["4,1,4,1,1", "2,2,2,2,1", "r,1,1,8", "r,2,2,4"]),
           ("bwd", "CONVMI_IGEMM_SPLIT", ["4,1,2,1,1,1,0", "4,1,2,1,1,1,1", "r,1,1,4,0", "r,2,1,8,1"]),
           ("upd", "CONVMI_UPD_SPLIT", ["1,2,2,2,2,16,16", "3,1,1,2,2,32,64"])]


@pytest.mark.parametrize("which,switch,variants", SPECIAL, ids=["fwd", "bwd", "upd"])
def test_infinities_and_nan_as_on_the_fp32_instructions(which, switch, variants):
    """... and values that round to infinity in bf16, of either sign."""
    shape = (2, 40, 48, 12, 13, 3, 3, 1, 1)
    I, Wt, dO = make_inputs(shape, F32, layer_id=54)
    rng = np.random.default_rng(8)
    for t in (I, Wt, dO):
        flat = t.reshape(-1)
        at = rng.choice(flat.size, 5, replace=False)
        flat[at] = [np.inf, -np.inf, np.nan, 3.4e38, -3.4e38] if t is not Wt else [np.inf, np.nan, 3.4e38, 1e-3, 1e-3]
    kw = {"fwd": dict(I=I, Wt=Wt), "bwd": dict(dO=dO, Wt=Wt), "upd": dict(I=I, dO=dO)}[which]
    got = []
    for v in ["0"] + variants:
        L = _layer(shape, **{switch: v})
        try:
            on = " on_bf16x3=" in conv.conv_describe(L.h, {"fwd": 0, "bwd": 1, "upd": 2}[which])
            assert on == (v != "0"), v
            got.append(run_pass(L, which, **kw).astype(np.float64))
        finally:
            L.close()
    fine = np.isfinite(got[0])
    assert 0.05 < fine.mean() < 1 and np.isinf(got[0]).any() and np.isnan(got[0]).any()
    for g, v in zip(got[1:], variants):
        assert np.array_equal(np.isfinite(g), fine), v
        assert np.array_equal(g[~fine], got[0][~fine], equal_nan=True), v
        small = fine & (np.abs(got[0]) < 1e30)
        assert_close(np.where(small, g, 0), np.where(small, got[0], 0), F32, v)


@pytest.mark.parametrize("which,switch,variants", SPECIAL, ids=["fwd", "bwd", "upd"])
@pytest.mark.parametrize("exponents", [(-60, -50), (-50, -48), (-108, 0), (-118, 10), (100, -20), (-116, 40), (-120, 50), (-124, 50)], ids=str)
def test_scale_does_not_matter(which, switch, variants, exponents):
    """Operands and results near and below the smallest bf16 numbers: powers of two times the operands give the same error (the fp32
    instructions round a product of 2^-110 and less to fewer bits too, and operands of 2^-124 are denormal from 2^-2 of the mean on,
    so not below that).  The scaled operands are rounded to fp32 first, and the reference is theirs."""
    shape = (2, 40, 48, 12, 13, 3, 3, 1, 1)
    I, Wt, dO = make_inputs(shape, F32, layer_id=55)
    a, b = {"fwd": (I, Wt), "bwd": (dO, Wt), "upd": (I, dO)}[which]
    refs = {"fwd": lambda: oracle.fwd(I, Wt, 1, 1), "bwd": lambda: oracle.bwd_data(dO, Wt, 12, 13, 1, 1), "upd": lambda: oracle.upd(I, dO, 3, 3, 1, 1)}
    for x, e in zip((a, b), exponents):  # (in place: what is left of it in fp32, scaled back for the oracle)
        x[...] = np.ldexp(np.ldexp(x, e).astype(np.float32).astype(np.float64), -e)
    ref = refs[which]()
    a *= np.float32(2.0 ** exponents[0])
    b *= np.float32(2.0 ** exponents[1])
    scale = 2.0 ** -(exponents[0] + exponents[1])
    kw = {"fwd": dict(I=I, Wt=Wt), "bwd": dict(dO=dO, Wt=Wt), "upd": dict(I=I, dO=dO)}[which]
    for v in variants:
        L = _layer(shape, **{switch: v})
        try:
            assert rel_l2(run_pass(L, which, **kw).astype(np.float64) * scale, ref) < 1e-6, v
        finally:
            L.close()


@pytest.mark.parametrize("which,switch,variants", SPECIAL, ids=["fwd", "bwd", "upd"])
@pytest.mark.parametrize("exponents", [(-60, -50), (-64, -60), (-70, -62), (-72, -68)], ids=str)
def test_tiny_sums_are_no_less_exact_than_on_the_fp32_instructions(which, switch, variants, exponents):
    """Sums whose small products are denormal numbers, and that are denormal themselves: the bf16 instructions keep such numbers."""
    shape = (2, 40, 48, 12, 13, 3, 3, 1, 1)
    I, Wt, dO = make_inputs(shape, F32, layer_id=58)
    ref = {"fwd": lambda: oracle.fwd(I, Wt, 1, 1), "bwd": lambda: oracle.bwd_data(dO, Wt, 12, 13, 1, 1), "upd": lambda: oracle.upd(I, dO, 3, 3, 1, 1)}[which]()
    a, b = {"fwd": (I, Wt), "bwd": (dO, Wt), "upd": (I, dO)}[which]
    a *= np.float32(2.0 ** exponents[0])  # (exact)
    b *= np.float32(2.0 ** exponents[1])
    kw = {"fwd": dict(I=I, Wt=Wt), "bwd": dict(dO=dO, Wt=Wt), "upd": dict(I=I, dO=dO)}[which]
    err = {}
    for v in ["0"] + variants:
        L = _layer(shape, **{switch: v})
        try:
            err[v] = rel_l2(np.ldexp(run_pass(L, which, **kw).astype(np.float64), -sum(exponents)), ref)
        finally:
            L.close()
    print(which, exponents, err, flush=True)
    assert all(e <= 1.1 * err["0"] for e in err.values()), err


@pytest.mark.parametrize("which,switch,variants", SPECIAL, ids=["fwd", "bwd", "upd"])
def test_tiny_values_among_others(which, switch, variants):
    """One channel of 2^-120 beside ordinary ones, in either operand, one that only another's 2^60 brings back, and sums of 2^-120 beside
    others of 2^-50: every channel of the result is as exact as in a tensor of its own.  And values between 2^-108 and 2^-107, whose
    last bf16 numbers are denormal."""
    shape = (2, 40, 48, 12, 13, 3, 3, 1, 1)
    rng = np.random.default_rng(11)
    I, Wt, dO = make_inputs(shape, F32, layer_id=57)
    few = 2.0 ** -108 * rng.uniform(1, 2, I.shape)
    tiny = np.float32(2.0 ** -120)
    cases = []
    for kind in ("a row", "a term", "a sum", "denormal parts"):
        x, w, g = I.copy(), Wt.copy(), dO.copy()
        if kind == "denormal parts":
            x = few.astype(np.float32)
            g = (2.0 ** -108 * rng.uniform(1, 2, dO.shape)).astype(np.float32)
            if which == "upd":
                g = (dO * np.float32(2.0 ** 40)).astype(np.float32)
            w *= np.float32(2.0 ** 40)
        elif kind == "a sum":  # (of operands that lose nothing; its small products are denormal)
            x *= np.float32(2.0 ** -50)
            g *= np.float32(2.0 ** -50)
            w[5] *= np.float32(2.0 ** -70)
            w[:, 7] *= np.float32(2.0 ** -70)
            if which == "upd":
                g = dO.copy()
                g[:, 5] *= np.float32(2.0 ** -70)
        elif kind == "a row":  # (of the result: a channel of its weights, or of dO, or of the input)
            w[5] *= tiny
            w[:, 7] *= tiny
            if which == "upd":
                x[:, 7] *= tiny
                g[:, 5] *= tiny
        else:  # (a term of every sum of a row, the others zero)
            x[:, 3] *= tiny
            g[:, 3] *= tiny
            w[9] = 0
            w[9, 3] = Wt[9, 3] * np.float32(2.0 ** 60)
            w[:, 9] = 0
            w[3, 9] = Wt[3, 9] * np.float32(2.0 ** 60)
            if which == "upd":
                g[:, 9] *= np.float32(2.0 ** 60)
        cases.append((kind, x, w, g))
    for kind, x, w, g in cases:
        X, W, G = (torch.from_numpy(t).double() for t in (x, w, g))
        if which == "fwd":
            ref, kw = torch.nn.functional.conv2d(X, W, padding=1), dict(I=x, Wt=w)
        elif which == "bwd":
            ref, kw = torch.nn.grad.conv2d_input(X.shape, W, G, padding=1), dict(dO=g, Wt=w)
        else:
            ref, kw = torch.nn.grad.conv2d_weight(X, W.shape, G, padding=1), dict(I=x, dO=g)
        per_channel = lambda t: np.sqrt(np.square(np.moveaxis(t, 1, 0).reshape(t.shape[1], -1) * 2.0 ** 60).sum(1)) + 1e-300
        rows = lambda t: np.sqrt(np.square(t.reshape(t.shape[0], -1) * 2.0 ** 60).sum(1)) + 1e-300
        for v in variants:
            L = _layer(shape, **{switch: v})
            try:
                d = run_pass(L, which, **kw).astype(np.float64) - ref.numpy()
            finally:
                L.close()
            for norm in (per_channel, rows) if which == "upd" else (per_channel,):
                assert (norm(d) <= 1e-6 * norm(ref.numpy())).all(), (kind, v, (norm(d) / norm(ref.numpy())).max())


# Where sums formed again meet strides, sampled pixels, cells of zeros, residue classes, strips and two sets of waves
AGAIN = [((3, 36, 52, 15, 13, 1, 1, 2, 0), "fwd", ["4,1,4,1,2,1", "2,2,2,2,1,1", "r,1,1,8"]), ((3, 36, 52, 15, 13, 1, 1, 2, 0), "upd", ["1,2,1,4,2,16,16", "1,1,1,2,2,64,64"]),
         ((3, 36, 52, 15, 13, 1, 1, 2, 0), "bwd", ["4,1,2,1,1,1,0", "2,2,2,2,1,1,1", "r,1,1,4,0", "r,2,2,4,1"]),
         ((2, 40, 36, 13, 12, 3, 3, 2, 1), "fwd", ["4,1,2,2,1,2", "2,2,4,1,1,1", "r,2,1,4"]), ((2, 40, 36, 13, 12, 3, 3, 2, 1), "bwd", ["4,1,4,1,1,1", "4,1,2,2,1,1", "2,2,2,1,1,1"]),
         ((2, 40, 36, 13, 12, 3, 3, 2, 1), "upd", ["3,1,1,2,4,16,64", "1,1,2,2,2,32,32"]), ((2, 36, 40, 9, 21, 1, 7, 1, (0, 3)), "fwd", ["4,1,2,1,1,3", "r,1,2,4"]),
         ((2, 36, 40, 9, 21, 1, 7, 1, (0, 3)), "bwd", ["2,2,2,2,1,2,1", "r,2,2,8,1"]), ((2, 36, 40, 9, 21, 1, 7, 1, (0, 3)), "upd", ["4,1,1,2,2,32,64", "5,1,1,2,2,16,32"])]


@pytest.mark.parametrize("kind", ["all NaN", "one NaN", "lost bits"])
@pytest.mark.parametrize("shape,which,variants", AGAIN, ids=lambda s: s if isinstance(s, str) else "x".join(map(str, s)).replace(" ", "") if isinstance(s, tuple) else "")
def test_sums_formed_again_under_every_geometry(shape, which, variants, kind):
    """Operands of 2^-120 that meet 2^50 against the oracle, and NaN (of one value, or of all) where the fp32 instructions have them."""
    N, C, K, H, W, R, S, stride, pad = shape
    I, Wt, dO = make_inputs(shape, F32, layer_id=59)
    a, b = {"fwd": (I, Wt), "bwd": (dO, Wt), "upd": (I, dO)}[which]
    switch = "CONVMI_UPD_SPLIT" if which == "upd" else "CONVMI_IGEMM_SPLIT"
    if kind == "lost bits":
        a[...] = np.ldexp(np.ldexp(a, -120).astype(np.float32).astype(np.float64), 120)  # (what is left of it in fp32)
        ref = {"fwd": lambda: oracle.fwd(I, Wt, stride, pad), "bwd": lambda: oracle.bwd_data(dO, Wt, H, W, stride, pad),
               "upd": lambda: oracle.upd(I, dO, R, S, stride, pad)}[which]()
        a *= np.float32(2.0 ** -120)
        b *= np.float32(2.0 ** 50)
    elif kind == "all NaN":
        a[...] = np.nan
    else:
        a.reshape(-1)[a.size // 2 + 3] = np.nan
    kw = {"fwd": dict(I=I, Wt=Wt), "bwd": dict(dO=dO, Wt=Wt), "upd": dict(I=I, dO=dO)}[which]
    got = {}
    for v in ["0"] + variants:
        L = _layer(shape, **{switch: v})
        try:
            assert (" on_bf16x3=" in conv.conv_describe(L.h, {"fwd": 0, "bwd": 1, "upd": 2}[which])) == (v != "0"), v
            print(shape, which, v, kind, flush=True)
            got[v] = run_pass(L, which, **kw).astype(np.float64)
        finally:
            L.close()
    for v in variants:
        if kind == "lost bits":
            assert_close(np.ldexp(got[v], 70), ref, F32, v)
        else:
            nan = np.isnan(got["0"])
            assert np.array_equal(np.isnan(got[v]), nan), v
            if np.where(nan, 0, got["0"]).any():
                assert_close(np.where(nan, 0, got[v]), np.where(nan, 0, got["0"]), F32, v)
            else:  # (all NaN but the cells of zeros)
                assert not np.where(nan, 0, got[v]).any(), v


# Layer, pass: relative error (2-norm) against 64 bits of what the planner picks, no larger than on the fp32 instructions
EXACT = [((28, 128, 128, 28, 28, 3, 3, 1, 1), "fwd"), ((16, 512, 512, 7, 7, 3, 3, 1, 1), "bwd"), ((8, 1024, 256, 14, 14, 1, 1, 1, 0), "fwd"),
         ((28, 128, 128, 28, 28, 3, 3, 1, 1), "upd"), ((16, 256, 512, 28, 28, 1, 1, 2, 0), "upd"), ((32, 64, 64, 56, 56, 3, 3, 1, 1), "upd"),
         ((32, 192, 192, 17, 17, 1, 7, 1, (0, 3)), "bwd"), ((16, 256, 256, 28, 28, 3, 3, 2, 1), "bwd")]


@pytest.mark.parametrize("shape,which", EXACT, ids=lambda s: s if isinstance(s, str) else "x".join(map(str, s)).replace(" ", ""))
def test_no_less_exact_than_the_fp32_instructions(shape, which):
    N, C, K, H, W, R, S, stride, pad = shape
    pads = pad if isinstance(pad, tuple) else (pad, pad)
    I, Wt, dO = make_inputs(shape, F32, layer_id=56)
    x, w, g = (torch.from_numpy(t).double() for t in (I, Wt, dO))
    if which == "fwd":
        ref = torch.nn.functional.conv2d(x, w, stride=stride, padding=pads)
    elif which == "bwd":
        ref = torch.nn.grad.conv2d_input(x.shape, w, g, stride=stride, padding=pads)
    else:
        ref = torch.nn.grad.conv2d_weight(x, w.shape, g, stride=stride, padding=pads)
    kw = {"fwd": dict(I=I, Wt=Wt), "bwd": dict(dO=dO, Wt=Wt), "upd": dict(I=I, dO=dO)}[which]
    err = []
    for env in (dict(CONVMI_IGEMM_SPLIT="0", CONVMI_UPD_SPLIT="0"), {}):
        L = _layer(shape, **env)
        try:
            assert (" on_bf16x3=" in conv.conv_describe(L.h, {"fwd": 0, "bwd": 1, "upd": 2}[which])) == (not env)
            err.append(rel_l2(run_pass(L, which, **kw), ref.numpy()))
        finally:
            L.close()
    assert err[1] <= 1.1 * err[0], err  # (the spread between inputs)


def _structured(kind, rows, cols, n, rng):
    """Two factors, rows x n and cols x n, of sums over n: few random products, one product other than zero, or all alike (then
    what the products leave out adds up); mantissas just above one leave out the most."""
    if kind == "short":
        return rng.standard_normal((rows, n)), rng.standard_normal((cols, n))
    a = rng.uniform(1, 1.0078, (rows, 1 if kind == "constant" else n)) * np.ones((1, n))
    if kind == "constant":
        return a, rng.uniform(1, 1.0078, (cols, 1)) * np.ones((1, n))
    b = np.zeros((cols, n))
    b[np.arange(cols), rng.integers(n, size=cols)] = rng.uniform(1, 1.0078, cols)
    return a, b


@pytest.mark.parametrize("kind,n", [("short", 16), ("short", 64), ("constant", 16), ("constant", 64), ("constant", 256), ("single", 16), ("single", 256)])
@pytest.mark.parametrize("which", ["fwd", "bwd", "upd"])
def test_sums_with_nothing_to_average_out(which, kind, n):
    """The products that are not formed are at most what rounding a product to fp32 costs, 2^-24 (1 + 2^-9) of it, and no sum is
    less exact for it than on the fp32 instructions, but for one product alone: what is left out of that is m*l and l*m with m spread over
    2^-8 and l over 2^-17 of either sign, at most sqrt(2) 2^-25 / 3 = 1.41e-8 in the mean, beside its rounding."""
    rng = np.random.default_rng(17)
    rows, cols = (64, 64) if which == "upd" else (1024, 64)
    a, b = (x.astype(np.float32) for x in _structured(kind, rows, cols, n, rng))
    ref, mag = (f(a).astype(np.float64) @ f(b).astype(np.float64).T for f in (lambda x: x, np.abs))
    if which == "upd":  # a: input channels over pixels, b: output channels
        side = int(n ** 0.5)
        shape, variants, switch = (1, 64, 64, side, side, 1, 1, 1, 0), ["1,1,1,2,2,32,32,1", "1,2,2,2,2,16,16,1"], "CONVMI_UPD_SPLIT"
        kw = dict(I=a.reshape(1, 64, side, side), dO=b.reshape(1, 64, side, side))
        back = lambda g: g[:, :, 0, 0].T
    else:  # a: pixels, b: the result's channels
        shape = (1, n, cols, 32, 32, 1, 1, 1, 0) if which == "fwd" else (1, cols, n, 32, 32, 1, 1, 1, 0)
        variants, switch = ["4,1,4,1,1", "2,2,2,1,2", "r,1,1,4"], "CONVMI_IGEMM_SPLIT"
        x = np.ascontiguousarray(a.T).reshape(1, n, 32, 32)
        kw = dict(I=x, Wt=b.reshape(cols, n, 1, 1)) if which == "fwd" else dict(dO=x, Wt=np.ascontiguousarray(b.T).reshape(n, cols, 1, 1))
        back = lambda g: g[0].reshape(cols, -1).T
    err = {}
    for v in ["0"] + variants:
        L = _layer(shape, **{switch: v})
        try:
            assert (" on_bf16x3=" in conv.conv_describe(L.h, {"fwd": 0, "bwd": 1, "upd": 2}[which])) == (v != "0"), v
            got = back(run_pass(L, which, **kw)).astype(np.float64)
        finally:
            L.close()
        err[v] = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        # left out, and one rounding of the sum for sixteen products, the small ones' sum and the result
        roundings = 1 + (0 if kind == "single" else n / 16 + 1)
        if v != "0":
            assert (np.abs(got - ref) <= 2.0 ** -24 * ((1 + 2.0 ** -9) * mag + roundings * (1 + 2.0 ** -7) * mag)).all(), v
            assert err[v] <= (np.hypot(err["0"], 1.41e-8) if kind == "single" else err["0"]), (v, err)


def _time_us(run):
    run()
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return min(times)


SLOWEST = [((28, 128, 128, 28, 28, 3, 3, 1, 1), "fwd"), ((28, 128, 128, 28, 28, 3, 3, 1, 1), "bwd"), ((32, 512, 512, 7, 7, 3, 3, 1, 1), "fwd"),
           ((32, 512, 512, 7, 7, 3, 3, 1, 1), "bwd"), ((64, 512, 1024, 28, 28, 1, 1, 2, 0), "fwd"), ((64, 512, 1024, 28, 28, 1, 1, 2, 0), "bwd"),
           ((32, 512, 512, 7, 7, 3, 3, 1, 1), "upd"), ((64, 64, 64, 56, 56, 3, 3, 1, 1), "upd"), ((64, 512, 1024, 28, 28, 1, 1, 2, 0), "upd")]


@pytest.mark.parametrize("shape,which", SLOWEST, ids=lambda s: s if isinstance(s, str) else "x".join(map(str, s)))
def test_nan_and_tiny_tensors_take_no_multiple_of_the_fp32_instructions_time(shape, which):
    """Sums that the bf16 instructions cannot form are formed again on the fp32 instructions: both passes together, 2 to 3 times what the
    plan on the fp32 instructions takes; at most 4, against runs that differ.  (One product at a time it was 5 to 30.)  Sums of 2^-110 from
    operands that lose nothing are left as they are, 0.6 - 0.8 of its time (formed again, 2.1); at most 1.3."""
    took = {}
    for env in ("0", None):
        L = _layer(shape, **({} if env is None else dict(CONVMI_IGEMM_SPLIT=env, CONVMI_UPD_SPLIT=env)))
        try:
            assert (" on_bf16x3=" in conv.conv_describe(L.h, {"fwd": 0, "bwd": 1, "upd": 2}[which])) == (env is None)
            src = L.out_blk if which == "bwd" else L.in_blk
            for t in (L.in_blk, L.out_blk, L.wt_blk):
                t.normal_()
            run = {"fwd": L.fwd, "bwd": L.bwd_data, "upd": L.upd}[which]
            for kind in ("nan", "tiny", "tiny sums"):
                if kind == "tiny sums":
                    src.normal_().mul_(2.0 ** -60)
                    (L.out_blk if which == "upd" else L.wt_blk).normal_().mul_(2.0 ** -50)
                elif kind == "tiny":
                    src.normal_().mul_(1e-38)
                else:
                    src.fill_(float("nan"))
                took[env, kind] = _time_us(run)
        finally:
            L.close()
    for kind, most in (("nan", 4), ("tiny", 4), ("tiny sums", 1.3)):
        assert took[None, kind] < most * took["0", kind], took
    print(which, shape, took, flush=True)
