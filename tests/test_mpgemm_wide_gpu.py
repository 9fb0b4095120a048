"""The prefill kernel without a weight tile (256 rows x 96 tokens per workgroup), which the launcher takes where the rounds of
its grid fit better, and the K-split tiles around the ends of K: ragged rows and tokens, K of half a 64-column stage, of one
stage, of an odd number of stages, and the longest K, where eight waves share it."""
import contextlib

import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import TOL, dev, mpgemm, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu


TOL_I8 = 1e-3  # as in the tests of the int8 calls: fp32 scaling and one fp16 rounding behind exact integers


@contextlib.contextmanager
def _tiling(**fields):
    t = tman.tman_get_tiling()
    try:
        forced = tman.tman_get_tiling()
        for name, value in fields.items():
            setattr(forced, name, value)
        tman.tman_set_tiling(forced)
        yield
    finally:
        tman.tman_set_tiling(t)


def _tiled(shape, blob, x, row_blocks):
    with _tiling(prefill_row_blocks=row_blocks):
        assert tman.tman_mpgemm_splits_k(shape, x.shape[0]) == 0
        return mpgemm(shape, blob, x)


def _against_tiled(shape, blob, x, y):
    """Every output against the tiled kernel: the same products, sums in another order (fp32, then one rounding)."""
    other = _tiled(shape, blob, x, 2).astype(np.float64)
    rms = np.sqrt(np.mean(other ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - other) <= 2.0 ** -10 * np.maximum(np.abs(other), rms))


@pytest.mark.parametrize("M,K,bits,group,hz,N", [
    (21700, 160, 4, 32, True, 288),   # two and a half stages
    (21760, 32, 2, 32, True, 97),     # half a stage
    (21505, 64, 1, 64, False, 193),   # one stage; the last row block has one row
    (21760, 192, 1, 32, True, 285),   # three stages
    (21698, 384, 4, 128, True, 96),
    (21700, 96, 2, 32, True, 191),
])
def test_wide_tiles(oracle_lib, M, K, bits, group, hz, N):
    q, s, z, x = rand_case(8100 + M + K + bits + N, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    assert tman.tman_mpgemm_splits_k(shape, N) == 0 and tman.tman_mpgemm_tile_rows(shape, N) == 256
    blob = pack(shape, q, s, z)
    # the activations lie between values that are not finite: a product with what lies outside them would show (a product with the
    # next token's columns, which are what lies beyond a token's K, shows in test_a_token_that_is_not_finite_stays_alone)
    xbig = torch.full((512 + N * K + 70000,), float("nan"), dtype=torch.float16, device=dev())
    xbig[512:512 + N * K] = to_dev(x).reshape(-1)
    y = mpgemm(shape, blob, xbig[512:512 + N * K].view(N, K))
    assert np.all(np.isfinite(y.astype(np.float32)))
    tokens = np.unique([0, 31, 32, 95, N // 2, N - 1])
    assert oracle.row_relative_error(y[tokens], oracle.matmul(q, s, z, x[tokens], bits, group)).max() <= TOL
    _against_tiled(shape, blob, x, y)
    # That no tiled kernel ran (256 x 256 tiles are 256 rows without a split of K as well): those give the same bits whatever their
    # rows; this one sums 8 columns of each of two blocks at a time, so where fp32 sums of activations of many sizes are inexact, some
    # of two million round differently (not with one block alone, whose columns every kernel sums in the same order).
    if K > 32:
        x = np.ldexp(x, np.random.default_rng(K).integers(-10, 9, x.shape)).astype(np.float16)
        y, tiled = mpgemm(shape, blob, x), _tiled(shape, blob, x, 4)
        assert np.array_equal(tiled, _tiled(shape, blob, x, 2)) and np.any(tiled != y)


@pytest.mark.parametrize("M,K,bits,group,hz,N", [
    (130, 544, 4, 32, True, 70),      # eight and a half stages over four waves
    (64, 576, 2, 64, True, 64),       # nine stages
    (65, 608, 1, 32, False, 129),
    (100, 640, 1, 32, True, 40),
    (64, 8192, 4, 64, True, 65),      # eight waves, 16 stages each
    (70, 8224, 4, 32, True, 33),      # ... and half a stage
    (65, 11008, 2, 128, True, 100),
])
def test_k_split_ends_of_k(oracle_lib, M, K, bits, group, hz, N):
    q, s, z, x = rand_case(8500 + M + K + bits + N, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    assert tman.tman_mpgemm_splits_k(shape, N) == 1
    blob = pack(shape, q, s, z)
    y = mpgemm(shape, blob, x)
    assert oracle.row_relative_error(y, oracle.matmul(q, s, z, x, bits, group)).max() <= TOL
    _against_tiled(shape, blob, x, y)


# The tiled kernel asks for the activations of its first four stages ahead of the loop and around its first barrier, with one row
# block from two waves, half of the tokens each: K of one to nine stages, tokens on both sides of every wave's last.
@pytest.mark.parametrize("row_blocks", [1, 2, 3, 4])
@pytest.mark.parametrize("M,K,bits,group,N", [
    (70, 32, 4, 32, 128),
    (130, 64, 2, 64, 129),
    (200, 96, 1, 32, 256),
    (260, 128, 4, 128, 257),
    (70, 160, 2, 32, 391),
    (190, 192, 4, 64, 100),
    (64, 288, 1, 32, 300),
])
def test_tiled_first_stages(oracle_lib, row_blocks, M, K, bits, group, N):
    q, s, z, x = rand_case(8600 + M + K + bits + N, M, K, N, bits, group, True)
    shape = tman.Shape(M, K, bits, group, True)
    y = _tiled(shape, pack(shape, q, s, z), x, row_blocks)
    assert oracle.row_relative_error(y, oracle.matmul(q, s, z, x, bits, group)).max() <= TOL


# K is an odd multiple of 32: the stage of 64 columns that ends with it holds the next token's first 32 columns too
@pytest.mark.parametrize("M,K,bits,group,hz,N,forced,rows,splits_k", [
    (70, 96, 4, 32, True, 300, dict(prefill_row_blocks=1), 64, 0),       # tiled
    (130, 160, 2, 32, True, 257, dict(prefill_row_blocks=2), 128, 0),
    (192, 32, 1, 32, False, 40, dict(prefill_row_blocks=3), 192, 0),
    (250, 352, 4, 32, True, 300, dict(prefill_row_blocks=4), 256, 0),
    (100, 544, 4, 32, True, 270, dict(prefill_k_split=2), 64, 1),        # K split, 64 x 256
    (130, 160, 1, 32, True, 130, dict(prefill_k_split=3), 128, 1),       # ... 128 x 128
    (8256, 1056, 4, 32, True, 97, {}, 64, 1),                            # ... 64 x 128
    (130, 544, 2, 32, True, 70, {}, 64, 1),                              # ... 64 x 64, four waves
    (70, 8224, 4, 32, True, 33, {}, 64, 1),                              # ... eight waves
    (21700, 160, 4, 32, True, 288, {}, 256, 0),                          # without a weight tile
    (21760, 32, 2, 32, True, 97, {}, 256, 0),
])
def test_a_token_that_is_not_finite_stays_alone(M, K, bits, group, hz, N, forced, rows, splits_k):
    """An infinity and a NaN among a token's first 32 columns: what lies beyond the token before it is not multiplied."""
    q, s, z, x = rand_case(8700 + M + K + bits + N, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    bad = x.copy()
    nan, inf = [1, N - 1], [N // 2]
    bad[nan, 5], bad[inf, 31] = np.nan, np.inf
    with _tiling(**forced):
        assert tman.tman_mpgemm_tile_rows(shape, N) == rows and tman.tman_mpgemm_splits_k(shape, N) == splits_k
        y, got = mpgemm(shape, blob, x), mpgemm(shape, blob, bad)
    assert np.all(np.isnan(got[nan])) and not np.any(np.isfinite(got[inf]))
    others = np.setdiff1d(np.arange(N), nan + inf)
    assert np.all(np.isfinite(y.astype(np.float32))) and np.array_equal(got[others], y[others])


# M that is no multiple of 8: words where it is even and y allows them, elements otherwise; the last row tile of one row, two, or all but
# one, the last token tile of one token or full
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("M,N,forced", [
    (65, 257, dict(prefill_row_blocks=1)),
    (130, 256, dict(prefill_row_blocks=2)),
    (383, 300, dict(prefill_row_blocks=3)),
    (514, 257, dict(prefill_row_blocks=4)),
    (21700, 97, {}),                          # without a weight tile
    (21505, 192, {}),
    (129, 129, dict(i8_token_blocks=1)),
    (258, 97, dict(i8_token_blocks=3)),
    (511, 128, dict(i8_token_blocks=4)),
    (257, 225, dict(i8_token_blocks=7)),
    (65, 300, dict(prefill_k_split=2)),
    (255, 129, dict(prefill_k_split=3)),
    (8258, 97, dict(K=1056)),                 # K split, 64 x 128
    (127, 70, dict(K=544)),                   # ... 64 x 64
    (65, 33, dict(K=8224)),                   # ... eight waves
    (258, 193, dict(i8_token_blocks=9)),
])
def test_rows_of_y_that_are_not_aligned(M, N, forced, offset):
    """The bits of the same rows among M rounded up to a multiple of 8, and nothing written beside them."""
    splits = 0 if not forced else 1 if "K" in forced else None
    forced = dict(forced)
    K, bits, group = forced.pop("K", 160), 4, 32
    full = (M + 7) // 8 * 8
    q, s, z, x = rand_case(9300 + M + N, full, K, N, bits, group)
    integer = "i8_token_blocks" in forced
    if integer:
        s, z = np.repeat(s[:, :1], K // group, axis=1), np.repeat(z[:, :1], K // group, axis=1)
    xd = to_dev(x)
    xq = torch.empty(tman.tman_act_i8_bytes(N, K), dtype=torch.uint8, device=dev())
    tman.tman_quantize_act_i8(xd, N, K, xq)

    def run(rows, y):
        shape = tman.Shape(rows, K, bits, group)
        blob = pack(shape, q[:rows], s[:rows], z[:rows])
        if splits is not None:
            assert (tman.tman_mpgemm_splits_k(shape, N), tman.tman_mpgemm_tile_rows(shape, N)) == ((1, 64) if splits else (0, 256))
        if integer:
            tman.tman_mpgemm_i8(shape, blob, xq, N, y, None)
        else:
            tman.tman_mpgemm(shape, blob, xd, N, y, None)
        torch.cuda.synchronize()

    room = torch.full((N * M + 24,), 777.0, dtype=torch.float16, device=dev())
    whole = torch.empty((N, full), dtype=torch.float16, device=dev())
    with _tiling(**forced):
        run(M, room[8 + offset:8 + offset + N * M])
        run(full, whole)
    got, mark = room.cpu().numpy().view(np.uint16), np.float16(777.0).view(np.uint16)
    assert np.all(got[:8 + offset] == mark) and np.all(got[8 + offset + N * M:] == mark)
    assert np.array_equal(got[8 + offset:8 + offset + N * M].reshape(N, M), whole.cpu().numpy()[:, :M].view(np.uint16))


@pytest.mark.parametrize("blocks", [1, 3, 4, 7, 9])
@pytest.mark.parametrize("M,K,bits,group,hz,N", [
    (70, 160, 4, 32, True, 100),      # a tile and a quarter
    (300, 1056, 2, 32, True, 230),    # nine tiles, the last with one block
    (257, 640, 1, 64, False, 129),    # five tiles: the loop of two runs one past the end
    (64, 2304, 4, 128, True, 33),     # 18 tiles over four waves
])
def test_int8_kernels_give_the_same_bits(oracle_lib, blocks, M, K, bits, group, hz, N):
    q, s, z, x = rand_case(8900 + M + K + bits + N, M, K, N, bits, group, hz)
    s = np.repeat(s[:, :1], K // group, axis=1)
    z = np.repeat(z[:, :1], K // group, axis=1) if hz else None
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    xq = torch.empty(tman.tman_act_i8_bytes(N, K), dtype=torch.uint8, device=dev())
    tman.tman_quantize_act_i8(to_dev(x), N, K, xq)
    codes, step = oracle.quantize_activations_i8(x)

    def run(kernel, acc):
        y = torch.full((N, M), float("nan"), dtype=torch.float16, device=dev())
        with _tiling(i8_token_blocks=kernel):
            tman.tman_mpgemm_i8(shape, blob, xq, N, y, acc)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    acc = torch.full((N, M), -1, dtype=torch.int32, device=dev())
    y = run(blocks, acc)
    want, Y = oracle.matmul_i8(q, s[:, 0], z[:, 0] if hz else None, codes, step, bits)
    assert np.array_equal(acc.cpu().numpy(), want)
    assert np.all(np.isfinite(y.astype(np.float32))) and oracle.row_relative_error(y, Y).max() <= TOL_I8
    # the sums are integers, so every kernel scales the same numbers: the same bits, with and without the sums as an output
    assert np.array_equal(y, run(blocks, None)) and np.array_equal(y, run(1, None))
