"""Chains in which the partial copies of dW are summed: 32 of them take a work-item per 16 bytes of dW and chain, which
passes the 2^32 work-items of a dispatch from 2 GiB of dW on.  Host only: the plan of an update in many chunks."""
import pytest

from paper_1808_05567_amd import conv

# N (images, one to a chunk), C = K, filter; chains
CASES = [(65, 64, 3, 32), (64, 64, 3, 8), (8, 64, 3, 1), (70, 7680, 3, 32), (70, 7936, 3, 8), (70, 8192, 3, 8), (8, 8192, 3, 1),
         (70, 15000, 3, 8)]


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
