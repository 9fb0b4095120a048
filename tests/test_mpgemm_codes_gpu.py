"""The small-batch kernel that multiplies codes and applies scales and zeros to the sums of quantization blocks: precision at
its token ranges, K edges inside a tile, segments, infinities and NaN."""
import numpy as np
import pytest

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import mpgemm, pack, rand_case

pytestmark = pytest.mark.gpu

FORMATS = [(1, True), (1, False), (2, True), (4, True)]


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group,N", [(32, 1), (32, 8), (64, 2), (64, 9), (64, 16), (128, 7), (128, 16), (128, 17), (128, 32)])
@pytest.mark.parametrize("M,K", [(65, 128), (40, 160), (70, 4096), (33, 5664)])
def test_sums_of_codes(oracle_lib, M, K, group, bits, hz, N):
    """The weights are not rounded, so what is left is the fp16 result, 2^-11 of the value, and the fp32 sums of
    (offset + c) x inside a block: normal x keep their partial sums below 80 * 4 * sqrt(128) = 3600 (offset 64, 4 bits),
    each of up to 16 additions rounds by 2^-24 of that, 3.4e-3 if all fell to one side, against sums of (c - z) x of
    rms 52: less than 1e-4 of rms(y) (the other formats have offsets of 4 and 2)."""
    K = -(-K // group) * group
    q, s, z, x = rand_case(6100 + M + K + bits + N + group, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    Y = oracle.matmul(q, s, z, x, bits, group)
    y = mpgemm(shape, pack(shape, q, s, z), x).astype(np.float64)
    rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) * 1.001 + 1e-4 * rms)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group,N", [(32, 3), (64, 12), (128, 20)])
def test_infinities_and_nan(oracle_lib, group, N, bits, hz):
    M, K = 66, 5760  # two segments; the values below lie in both, one token has none
    q, s, z, x = rand_case(6500 + bits, M, K, N, bits, group, hz)
    w = ((2.0 * q - 1.0) if z is None else q - z.astype(np.float64).repeat(group, axis=1)) * s.astype(np.float64).repeat(group, axis=1)
    x[0, 5], x[0, 5759] = np.inf, -np.inf
    x[1, 4097] = np.inf
    if N > 3:
        x[2, 131] = np.nan
        x[N - 1, 2000] = -np.inf
    shape = tman.Shape(M, K, bits, group, hz)
    with np.errstate(invalid="ignore"):
        ref = np.stack([(w * xi.astype(np.float64)).sum(axis=1) for xi in x])
    y = mpgemm(shape, pack(shape, q, s, z), x).astype(np.float64)
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref).all(axis=1)
    assert oracle.row_relative_error(y[ok], ref[ok]).max() <= 1e-3


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group,N", [(32, 8), (64, 16), (128, 32)])
def test_one_bad_sequence_leaves_the_others_alone(oracle_lib, group, N, bits, hz):
    """The tokens without infinities come out with the same bits as in a batch that has none."""
    M, K = 66, 5760  # two segments
    q, s, z, x = rand_case(6700 + bits, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    clean = mpgemm(shape, blob, x)
    x[1, 70], x[1, 5000] = np.inf, np.nan
    y = mpgemm(shape, blob, x)
    assert np.isnan(y[1].astype(np.float64)).all()
    others = np.arange(N) != 1
    assert np.array_equal(y[others].view(np.uint16), clean[others].view(np.uint16))


def test_next_token_does_not_leak_through_the_last_tile(oracle_lib):
    """K ends inside a tile: the columns beyond it are the next token's in memory."""
    M, K, bits, group, N = 64, 160, 4, 32, 4
    q, s, z, x = rand_case(6600, M, K, N, bits, group)
    x[1:] = 60000.0  # finite, but 1e5 times the first token's
    shape = tman.Shape(M, K, bits, group)
    y = mpgemm(shape, pack(shape, q, s, z), x)
    assert oracle.row_relative_error(y[:1], oracle.matmul(q, s, z, x[:1], bits, group)).max() <= 1e-3
