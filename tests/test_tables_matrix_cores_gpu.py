"""Two to eight tokens out of fp16 and integer tables on the matrix cores (and, few planes, by lookups): every padded token
count, K edges inside a tile, segments, infinities in one token, workspaces of the queried size."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import TOL, dev, gemv_workspace, mpgemv, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu

FORMATS = [(1, 64, True), (1, 32, False), (2, 32, True), (2, 128, True), (4, 32, True), (4, 64, True), (4, 128, True)]


def _integer(shape, blob, x):
    N, K = x.shape
    lut = torch.empty(tman.tman_lut_i16_bytes(N, K, shape.group), dtype=torch.uint8, device=dev())
    y = torch.full((N, shape.M), float("nan"), dtype=torch.float16, device=dev())
    tman.tman_build_lut_i16(to_dev(x), N, K, shape.group, lut)
    tman.tman_mpgemv_i16(shape, blob, lut, N, y, gemv_workspace(shape, N))
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("bits,group,hz", FORMATS)
@pytest.mark.parametrize("N", [2, 3, 5, 8])
@pytest.mark.parametrize("M,K", [(64, 128), (33, 192), (65, 1056), (70, 5632)])
def test_tables(oracle_lib, M, K, N, bits, group, hz, integer):
    """Activations that are multiples of the tokens' integer steps, so both kinds of tables hold them exactly: what is left is
    the fp16 result, 2^-11 of the value, and fp32 sums whose partial sums stay below 64 (the offset of a code) times the
    block's sum of x, at most 16 roundings of 2^-24 of that: below 1e-4 of rms(y).  (Lookups round table entries: TOL.)"""
    K = -(-K // group) * group
    q, s, z, _ = rand_case(9100 + M + K + N + bits, M, K, 1, bits, group, hz)
    x = np.random.default_rng(M + K + N).integers(-1023, 1024, size=(N, K)).astype(np.float16)
    x[:, 0] = 1023
    shape = tman.Shape(M, K, bits, group, hz)
    Y = oracle.matmul(q, s, z, x, bits, group)
    blob = pack(shape, q, s, z)
    y = (_integer(shape, blob, x) if integer else mpgemv(shape, blob, x)).astype(np.float64)
    if bits == 4 or N > 4:
        rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
        assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) * 1.001 + 1e-4 * rms)
    else:
        assert oracle.row_relative_error(y, Y).max() <= TOL


@pytest.mark.parametrize("bits,group,N", [(4, 128, 2), (4, 32, 8), (2, 64, 3), (1, 64, 7)])
def test_infinities_in_one_token(oracle_lib, bits, group, N):
    M, K = 66, 5760  # two segments
    q, s, z, x = rand_case(9300 + bits, M, K, N, bits, group)
    shape = tman.Shape(M, K, bits, group)
    blob = pack(shape, q, s, z)
    clean = mpgemv(shape, blob, x)
    x[1, 70], x[1, 5000] = np.inf, -np.inf
    w = (q - z.astype(np.float64).repeat(group, axis=1)) * s.astype(np.float64).repeat(group, axis=1)
    with np.errstate(invalid="ignore"):
        ref = (w * x[1].astype(np.float64)).sum(axis=1)
    y = mpgemv(shape, blob, x)
    assert np.array_equal(np.isnan(y[1]), np.isnan(ref)) and np.array_equal(y[1][np.isinf(ref)].astype(np.float64), ref[np.isinf(ref)])
    others = np.arange(N) != 1
    assert np.array_equal(y[others].view(np.uint16), clean[others].view(np.uint16))
