"""One token with 1- and 2-bit weights on the matrix cores: the split of an activation into four 8-bit numbers (every exponent), the
sums at edges of tiles and row blocks, activations as such and out of tables."""
import numpy as np
import pytest

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import mpgemv, mpgemv_x, pack, rand_case

pytestmark = pytest.mark.gpu

FORMATS = [(1, True), (1, False), (2, True)]


def _repeat(a, group):
    return a.astype(np.float64).repeat(group, axis=1)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group,K", [(32, 160), (64, 192), (128, 256)])
def test_one_activation_of_every_exponent(oracle_lib, group, K, bits, hz):
    """With one activation that is not zero nothing is added to anything: the split has to be exact, the rest is one rounding each
    of z S, the difference, the scaling (2^-24 of s (q + |z|) |x|) and the fp16 result."""
    M = 70
    q, s, z, _ = rand_case(9700 + K, M, K, 1, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    rng = np.random.default_rng(K + bits)
    w = ((2.0 * q - 1.0) if z is None else q - _repeat(z, group)) * _repeat(s, group)
    size = ((2.0 * q + 1.0) if z is None else q + np.abs(_repeat(z, group))) * _repeat(s, group)
    for exponent in range(31):
        k = int(rng.integers(0, K))
        x = np.zeros((1, K), dtype=np.uint16)
        x[0, k] = exponent << 10 | int(rng.integers(0, 1024)) | int(rng.integers(0, 2)) << 15
        x = x.view(np.float16)
        y = mpgemv_x(shape, blob, x).astype(np.float64).ravel()
        ref, terms = w[:, k] * float(x[0, k]), size[:, k] * abs(float(x[0, k]))
        assert np.all(np.abs(y - ref) <= 2.0 ** -11 * np.abs(ref) + 4 * 2.0 ** -24 * terms + 2.0 ** -25), exponent


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("M,K", [(1, 128), (64, 32), (65, 416), (130, 4096), (63, 5696)])
def test_sums(oracle_lib, M, K, group, bits, hz):
    """Normal activations.  They are rounded to 2^-18 of the power of two above the largest of their 32 columns, 4 (once in a while 8), to
    2^-16: less than 1e-4 of rms(y) beside the fp16 result."""
    K = -(-K // group) * group
    q, s, z, x = rand_case(9750 + M + K, max(M, 33), K, 1, bits, group, hz)
    shape = tman.Shape(max(M, 33), K, bits, group, hz)
    Y = oracle.matmul(q, s, z, x, bits, group)
    y = mpgemv_x(shape, pack(shape, q, s, z), x).astype(np.float64)
    rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) * 1.001 + 1e-4 * rms)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("one_sign", [False, True])
@pytest.mark.parametrize("group,outlier", [(32, 100), (32, 1000), (32, 4000), (64, 1000), (64, 4000), (128, 4000)])
def test_large_channels(oracle_lib, group, outlier, one_sign, bits, hz):
    """1 % of the channels up to 4000 times the others, also with activations of one sign, where errors of one sign would add up.
    What is left is the fp16 result (a step of the result, uniform: / sqrt(12)) and activations rounded to the step of their 32
    columns, 2^-18 of the power of two above the largest, to either side alike: the mean error of 1024 rows lies within five
    standard deviations of zero."""
    M, K = 1024, 4096
    q, s, z, _ = rand_case(9900 + bits + group, M, K, 1, bits, group, hz)
    rng = np.random.default_rng(outlier + group)
    x = rng.standard_normal(K)
    x[rng.permutation(K)[:K // 100]] *= outlier
    x = (np.abs(x) if one_sign else x).astype(np.float16).reshape(1, K)
    w = ((2.0 * q - 1.0) if z is None else q - _repeat(z, group)) * _repeat(s, group)
    xd = x[0].astype(np.float64)
    Y = w @ xd
    step = np.exp2(np.ceil(np.log2(np.abs(xd).reshape(-1, 32).max(axis=1))) - 18).repeat(32)
    rounded = np.rint(xd / step) != xd / step
    half = np.exp2(np.maximum(np.floor(np.log2(np.abs(Y) + 1e-30)), -14) - 10)
    expected = np.sqrt(np.mean(((w * w) @ np.where(rounded, step * step, 0.0) + half * half) / 12.0))
    shape = tman.Shape(M, K, bits, group, hz)
    error = mpgemv_x(shape, pack(shape, q, s, z), x)[0].astype(np.float64) - Y
    assert np.sqrt(np.mean(error ** 2)) <= 1.1 * expected
    assert abs(np.mean(error)) <= 5 * expected / np.sqrt(M)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("M,K,group", [(65, 416, 32), (70, 4160, 64)])
def test_activations_out_of_tables(oracle_lib, M, K, group, bits, hz):
    """Entries 1, 2, 4 and 8 of a table are the activations: the same bits as without tables."""
    q, s, z, x = rand_case(9800 + M, M, K, 1, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    assert np.array_equal(mpgemv(shape, blob, x).view(np.uint16), mpgemv_x(shape, blob, x).view(np.uint16))
