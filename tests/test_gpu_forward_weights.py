"""Backward by data reading the forward pass's weights in the staged kernel (every instantiation: a host test holds the
shapes here against the list of them), in the residue
classes of a strided pass and in the register-operand kernel, against the oracle at the edges: ragged channels both
ways (an odd number of channel blocks), one pixel, images smaller than a tile, tiles
that cross images, padding other than "same", the scattering store.  The workspace holds NaN patterns: nothing may be
read from it.  Bars: gpu_util.assert_close."""
import re

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
    # two, three and more staged positions per thread: long rows, many small images to a tile, tall narrow images
    (2, 40, 64, 5, 64, 3, 3, 1, 1),
    (70, 40, 64, 1, 2, 3, 3, 1, 1),
    (3, 72, 48, 60, 5, 3, 3, 1, 1),
    (3, 40, 64, 7, 8, 7, 1, 1, (3, 0)),
    (1, 40, 64, 7, 40, 7, 1, 1, (3, 0)),
]


def tiles(shape, dtype):
    return (TILES_1X1 if shape[5] * shape[6] == 1 else TILES)[dtype]


def staged_variant(tile, text):
    """The instantiation that a plan for `tile` runs on (type, waves, fragments, channel blocks, filter, positions per
    thread, buffers, input policy); None if it is another tile or transforms the weights."""
    wk, wm, fk, fm, nb, npl = tile.split(",")
    m = re.match(r"igemm dt=(\d) waves=%sx%s frags=%sx%s npl=(\d+) nt=(\d) RS=(\S+) ppt=(\d+) .*forward_weights=1"
                 % (wk, wm, fk, fm), text)
    return m and (int(m[1]), wk + "x" + wm, fk + "x" + fm, int(m[2]), m[4], int(m[5]), int(nb), int(m[3]))


@pytest.mark.parametrize("dtype", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_staged_tiles_match_oracle(shape, dtype, monkeypatch):
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, dtype, layer_id=11)
    ref = oracle.bwd_data(dO, Wt, H, W, stride, pad)
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    ran = set()
    for tile in tiles(shape, dtype):
        for nt in ("0", "1"):  # (the input non-temporally, where that is built)
            monkeypatch.setenv("CONVMI_IGEMM_CAND", tile)
            monkeypatch.setenv("CONVMI_IGEMM_NT", nt)
            L = conv.ConvLayer(*shape, dtype=dtype)
            try:
                v = staged_variant(tile, conv.conv_describe(L.h, conv.PASS_BWD_DATA))
                if v and v not in ran:
                    ran.add(v)
                    L.ws.fill_(0xFF)
                    assert_close(run_pass(L, "bwd", Wt=Wt, dO=dO), ref, dtype, tile)
            finally:
                L.close()
    assert len(ran) >= 2, ran


@pytest.mark.parametrize("shape,env", [
    ((5, 36, 48, 7, 8, 3, 3, 2, 0), ("CONVMI_BWD_QUAD", "1")),
    ((3, 100, 48, 13, 11, 3, 3, 2, 1), ("CONVMI_BWD_QUAD", "1")),
    ((3, 264, 160, 13, 11, 1, 1, 1, 0), ("CONVMI_IGEMM_CAND", "4,1,1,7,2,4")),
    ((3, 40, 192, 9, 10, 1, 1, 2, 0), ("CONVMI_IGEMM_CAND", "2,2,2,2,2,8")),
    ((3, 40, 96, 9, 11, 7, 1, 1, (3, 0)), ("CONVMI_IGEMM_CAND", "2,2,1,2,2,2")),
], ids=str)
def test_fp32_passes_in_both_forms_are_the_same(shape, env, monkeypatch):
    """Long launches transform the weights after all: the same sums, in the same order."""
    N, C, K, H, W, R, S, stride, pad = shape
    _, Wt, dO = make_inputs(shape, conv.CONV_F32, layer_id=11)
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    monkeypatch.setenv(*env)
    got = []
    for form in ("0", "1"):
        monkeypatch.setenv("CONVMI_FORWARD_WEIGHTS", form)
        L = conv.ConvLayer(*shape, dtype=conv.CONV_F32)
        try:
            assert ("forward_weights=1" in conv.conv_describe(L.h, conv.PASS_BWD_DATA)) == (form == "1")
            L.ws.fill_(0xFF)
            got.append(run_pass(L, "bwd", Wt=Wt, dO=dO))
        finally:
            L.close()
    assert_close(got[0], oracle.bwd_data(dO, Wt, H, W, stride, pad), conv.CONV_F32, str(env))
    assert (got[0] == got[1]).all()


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
