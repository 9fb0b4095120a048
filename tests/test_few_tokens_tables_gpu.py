"""Two to eight tokens out of tables with 4-bit weights (the matrix cores multiply the codes): integer tables for every token count,
fp16 tables for two, K edges, the default segments and one segment of any length, infinities."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import dev, gemv_workspace, mpgemv, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu


def _i16(shape, blob, x):
    N, K = x.shape
    lut = torch.empty(tman.tman_lut_i16_bytes(N, K, shape.group), dtype=torch.uint8, device=dev())
    y = torch.full((N, shape.M), float("nan"), dtype=torch.float16, device=dev())
    tman.tman_build_lut_i16(to_dev(x), N, K, shape.group, lut)
    tman.tman_mpgemv_i16(shape, blob, lut, N, y, gemv_workspace(shape, N))
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


@pytest.fixture(params=[0, 100])
def seg_tiles(request):
    """0: the default segments; 100: one segment for every K here."""
    saved = tman.tman_get_tiling()
    if request.param:
        t = tman.tman_get_tiling()
        t.decode_seg_tiles = t.decode_seg_tiles_many = request.param
        tman.tman_set_tiling(t)
    yield request.param
    tman.tman_set_tiling(saved)


@pytest.mark.parametrize("N", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("M,K,group", [(65, 128, 128), (40, 160, 32), (33, 3200, 64), (70, 8320, 64), (64, 11008, 128)])
def test_integer_tables(oracle_lib, seg_tiles, M, K, group, N):
    """Activations that are multiples of the tokens' integer steps: the block sums are exact, the rest is the fp32 sum over
    blocks (K / group additions of 2^-24 against partial sums taken as 64 times the rms) and half a step of the result."""
    q, s, z, _ = rand_case(7100 + M + K + N, M, K, 1, 4, group)
    x = np.random.default_rng(M + K + N).integers(-2047, 2048, size=(N, K)).astype(np.float16)
    x[:, 0] = 2047  # fixes the steps
    shape = tman.Shape(M, K, 4, group)
    Y = oracle.matmul(q, s, z, x, 4, group)
    y = _i16(shape, pack(shape, q, s, z), x)
    rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) + 64 * (K // group) * 2.0 ** -24 * rms)


@pytest.mark.parametrize("N", [5, 8])
@pytest.mark.parametrize("K", [2944, 3072, 9216])
def test_blocks_of_32_in_long_segments(oracle_lib, seg_tiles, K, N):
    """Blocks of 32 and 5 to 8 tokens (two rows of the product each): 23, 24 and 72 tiles."""
    test_integer_tables(oracle_lib, seg_tiles, 40, K, 32, N)


@pytest.mark.parametrize("M,K,group", [(65, 128, 128), (40, 160, 32), (70, 8320, 64)])
def test_two_tokens_from_fp16_tables(oracle_lib, seg_tiles, M, K, group):
    q, s, z, _ = rand_case(7300 + M + K, M, K, 1, 4, group)
    x = (np.random.default_rng(K).integers(-1023, 1024, size=(2, K)) / 512.0).astype(np.float16)
    shape = tman.Shape(M, K, 4, group)
    blob = pack(shape, q, s, z)
    Y = oracle.matmul(q, s, z, x, 4, group)
    y = mpgemv(shape, blob, x).astype(np.float64)
    rms = np.sqrt(np.mean(Y ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - Y) <= 2.0 ** -11 * np.abs(Y) + 64 * (K // group) * 2.0 ** -24 * rms)
    x[1, K - 1], x[1, 3] = np.inf, np.inf
    w = (q - z.astype(np.float64).repeat(group, axis=1)) * s.astype(np.float64).repeat(group, axis=1)
    with np.errstate(invalid="ignore"):
        ref = np.stack([(w * xi.astype(np.float64)).sum(axis=1) for xi in x])
    y = mpgemv(shape, blob, x).astype(np.float64)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    assert oracle.row_relative_error(y[:1], ref[:1]).max() <= 1e-3
