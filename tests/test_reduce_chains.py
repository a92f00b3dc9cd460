"""Chains in which the partial copies of dW are summed: 32 of them take a work-item per 16 bytes of dW and chain, which
passes the 2^32 work-items of a dispatch from 2 GiB of dW on (host only: the plan of an update in many chunks).  And the sums
themselves, at the smallest and largest number of copies of each number of chains, against the oracle."""
import pytest

import oracle
from paper_1808_05567_amd import conv

# N (images, one to a chunk), C = K, filter; chains
CASES = [(65, 64, 3, 32), (64, 64, 3, 16), (32, 64, 3, 16), (31, 64, 3, 8), (9, 64, 3, 8), (8, 64, 3, 1), (70, 7680, 3, 32),
         (70, 7936, 3, 16), (70, 8192, 3, 16), (8, 8192, 3, 1), (70, 15000, 3, 8)]


@pytest.mark.parametrize("N,C,R,chains", CASES)
def test_sum_of_the_chunks_fits_a_dispatch(N, C, R, chains):
    h = conv.conv_create_chunked(N, C, C, 4, 4, R, R, 1, 1, 1)
    try:
        dwt = conv.conv_query(h).dwt_bytes
        assert dwt == 4 * C * C * R * R
        text = conv.conv_describe(h, conv.PASS_UPD)
        assert text.endswith(" chunk_chains=%d" % chains), text
        assert dwt // 16 * chains < 2 ** 32
    finally:
        conv.conv_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("copies", [2, 8, 9, 31, 32, 33, 63, 64, 65, 257])
@pytest.mark.parametrize("C,K", [(20, 8), (32, 64)])
def test_sums_of_copies_match_oracle(C, K, copies):
    from gpu_util import assert_close, make_inputs, run_pass
    # (one image to a chunk: one copy of dW per image; dW of 160 and 2048 groups of four elements)
    shape = (copies, C, K, 5, 4, 1, 1, 1, 0)
    I, _, dO = make_inputs(shape, conv.CONV_F32, layer_id=37)
    L = conv.ConvLayer(*shape, dtype=conv.CONV_F32, max_images=1)
    try:
        chains = 1 if copies <= 8 else 8 if copies < 32 else 16 if copies <= 64 else 32
        assert conv.conv_describe(L.h, conv.PASS_UPD).endswith(" chunk_chains=%d" % chains)
        assert_close(run_pass(L, "upd", I=I, dO=dO), oracle.upd(I, dO, 1, 1, 1, 0), conv.CONV_F32, "upd")
    finally:
        L.close()
