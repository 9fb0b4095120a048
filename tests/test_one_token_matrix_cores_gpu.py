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
    """Normal activations.  Of 8 neighbouring products the matrix cores keep what is at least 2^-13 of the largest; a product is a code
    times a digit of 3 bits, so what is cut lies below 2^-11 (of activations up to 4) and comes from digits that small: less than
    1e-4 of rms(y) beside the fp16 result."""
    K = -(-K // group) * group
    q, s, z, x = rand_case(9750 + M + K, max(M, 33), K, 1, bits, group, hz)
    shape = tman.Shape(max(M, 33), K, bits, group, hz)
    Y = oracle.matmul(q, s, z, x, bits, group)
    y = mpgemv_x(shape, pack(shape, q, s, z), x).astype(np.float64)
    rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) * 1.001 + 1e-4 * rms)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("M,K,group", [(65, 416, 32), (70, 4160, 64)])
def test_activations_out_of_tables(oracle_lib, M, K, group, bits, hz):
    """Entries 1, 2, 4 and 8 of a table are the activations: the same bits as without tables."""
    q, s, z, x = rand_case(9800 + M, M, K, 1, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    assert np.array_equal(mpgemv(shape, blob, x).view(np.uint16), mpgemv_x(shape, blob, x).view(np.uint16))
