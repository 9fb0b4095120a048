"""The kernel that multiplies codes where quantization blocks share a product: blocks of 32 with 9 to 16 tokens (precision,
infinities), and a last tile whose columns beyond K are, in memory, the next token's."""
import numpy as np
import pytest

import oracle
import paper_2511_11248_amd as tman
import test_mpgemm_codes_gpu as codes
from gpu_helpers import mpgemm, pack, rand_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,hz", codes.FORMATS)
@pytest.mark.parametrize("N", [9, 16])
@pytest.mark.parametrize("M,K", [(65, 128), (40, 160), (33, 5664)])
def test_blocks_of_32(oracle_lib, M, K, N, bits, hz):
    codes.test_sums_of_codes(oracle_lib, M, K, 32, bits, hz, N)


@pytest.mark.parametrize("bits,hz", codes.FORMATS)
def test_blocks_of_32_with_infinities(oracle_lib, bits, hz):
    codes.test_infinities_and_nan(oracle_lib, 32, 13, bits, hz)
    codes.test_one_bad_sequence_leaves_the_others_alone(oracle_lib, 32, 13, bits, hz)


@pytest.mark.parametrize("group,K,N", [(32, 32, 2), (32, 160, 8), (32, 224, 16), (64, 64, 8), (64, 192, 5), (64, 320, 12)])
def test_next_token_infinite(oracle_lib, group, K, N):
    """The other tokens keep their sums when the columns behind theirs hold infinities."""
    q, s, z, x = rand_case(6900 + K, 70, K, N, 4, group)
    x[N - 1, :8] = np.inf
    shape = tman.Shape(70, K, 4, group)
    y = mpgemm(shape, pack(shape, q, s, z), x)[: N - 1]
    assert oracle.row_relative_error(y, oracle.matmul(q, s, z, x[: N - 1], 4, group)).max() <= 1e-3
