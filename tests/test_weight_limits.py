"""Weights whose bytes 32-bit offsets do not reach: conv_create takes up to 2^31 of them (8 GB in fp32), the
tiled forward and backward kernels address them with 32 bits, so such layers belong to the untiled loops, whose
indices are 64-bit.  Host only: the plans are described, nothing is launched."""
import pytest

from paper_1808_05567_amd import conv

F32, BF16 = conv.CONV_F32, conv.CONV_BF16

# N, C, K, H, W, R, S, stride, pad, type
BEYOND = [
    (1, 8192, 8192, 8, 8, 4, 4, 1, 1, F32),               # 4 GiB to the byte: a 32-bit size of zero
    (1, 5440, 5440, 20, 20, 7, 7, 1, 3, F32),             # 5.8 GB
    (1, 14680, 14680, 9, 9, 1, 5, 1, (0, 2), F32),        # 4.3 GB, a filter without a staged kernel
    (1, 32768, 32768, 7, 7, 1, 1, 1, 0, F32),             # 4 GiB, filters with staged kernels
    (1, 11264, 11264, 8, 8, 3, 3, 1, 1, F32),
    (1, 11264, 11264, 8, 8, 3, 3, 2, 1, F32),             # fwd 4.6 GB; its residue classes up to 2 GB each
    (1, 46000, 46000, 7, 7, 1, 1, 1, 0, BF16),            # 4.2 GB
]
WITHIN = [
    (1, 8192, 7424, 8, 8, 4, 4, 1, 1, F32),               # 3.9 GB
    (1, 31200, 31200, 7, 7, 1, 1, 1, 0, F32),
    (1, 44000, 44000, 7, 7, 1, 1, 1, 0, BF16),
]


def _describe(shape):
    h = conv.conv_create(*shape)
    try:
        return conv.conv_query(h).wt_bytes, [conv.conv_describe(h, p) for p in (conv.PASS_FWD, conv.PASS_BWD_DATA)]
    finally:
        conv.conv_destroy(h)


@pytest.mark.parametrize("shape", BEYOND, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_weights_beyond_32_bit_offsets_run_untiled(shape):
    wt_bytes, (fwd, bwd) = _describe(shape)
    assert wt_bytes > 4.0e9
    assert fwd.startswith("direct "), fwd
    assert "forward_weights=1" not in bwd, bwd
    if shape[7] == 1:  # (a strided pass transforms the weights into one sub-filter per residue class)
        assert bwd.startswith("direct "), bwd


@pytest.mark.parametrize("shape", WITHIN, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_weights_just_within_them_keep_their_tiled_kernels(shape):
    wt_bytes, plans = _describe(shape)
    assert 3.8e9 < wt_bytes <= 4.0e9
    assert all(p.startswith("igemm") for p in plans), plans


@pytest.mark.parametrize("shape", [
    (16, 12000, 12000, 28, 28, 3, 3, 2, 1, F32),          # 5.2 GB
    (8, 24000, 6000, 28, 28, 3, 3, 2, 1, F32),
    (8, 40000, 4000, 14, 14, 3, 3, 2, 1, F32),
    (8, 10800, 10400, 14, 14, 3, 3, 2, 1, F32),           # 4.04 GB
    (8, 15200, 15200, 14, 14, 3, 3, 2, 1, BF16),          # 4.2 GB
], ids=lambda s: "x".join(map(str, s)))
def test_strided_backward_of_such_weights_transforms_them(shape):
    """Each residue class is in reach, the whole filter is not: the classes run on their own, transformed weights."""
    wt_bytes, (fwd, bwd) = _describe(shape)
    assert wt_bytes > 4.0e9
    assert fwd.startswith("direct "), fwd
    assert bwd.startswith("igemm") and "forward_weights=1" not in bwd, bwd
    if shape[-1] == BF16:  # (no kernel for the classes in one launch reads transformed weights)
        assert "launches=4" in bwd, bwd


@pytest.mark.parametrize("shape", [(8, 10400, 10400, 14, 14, 3, 3, 2, 1, F32), (8, 14880, 14880, 14, 14, 3, 3, 2, 1, BF16)],
                         ids=lambda s: "x".join(map(str, s)))
def test_strided_backward_of_weights_just_within_reach_does_not(shape):
    wt_bytes, (fwd, bwd) = _describe(shape)
    assert 3.8e9 < wt_bytes <= 4.0e9
    assert fwd.startswith("igemm"), fwd
    if shape[-1] == BF16:  # (fp32: a launch of this length repays the transform)
        assert "launches=1" in bwd and "forward_weights=1" in bwd, bwd
