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
    """Activations that are multiples of the tokens' integer steps (1: the largest is 8184), so both kinds of tables hold them exactly;
    nine tenths take every rest modulo 8, which integer activations are split by.  What is left is
    the fp16 result, 2^-11 of the value, and fp32 sums whose partial sums stay below 64 (the offset of a code) times the
    block's sum of x, at most 16 roundings of 2^-24 of that: below 1e-4 of rms(y).  (Lookups round table entries: TOL.)"""
    K = -(-K // group) * group
    q, s, z, _ = rand_case(9100 + M + K + N + bits, M, K, 1, bits, group, hz)
    rng = np.random.default_rng(M + K + N)
    x = np.where(rng.random((N, K)) < 0.9, rng.integers(-2047, 2048, size=(N, K)), 8 * rng.integers(-1023, 1024, size=(N, K))).astype(np.float16)
    x[:, 0] = 8184
    shape = tman.Shape(M, K, bits, group, hz)
    Y = oracle.matmul(q, s, z, x, bits, group)
    blob = pack(shape, q, s, z)
    y = (_integer(shape, blob, x) if integer else mpgemv(shape, blob, x)).astype(np.float64)
    if bits == 4 or N > 4 or (bits == 2 and (N > 2 or integer)):
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


def _segments(shape, N, integer=False, batch=1):
    """K segments of a call with tables, by what it leaves in its workspace: behind the tickets, partial sums of every segment."""
    q, s, z, x = rand_case(9400 + N, shape.M, shape.K, N, shape.bits, shape.group)
    blob = pack(shape, q, s, z)
    size, build, one, many = ((tman.tman_lut_i16_bytes, tman.tman_build_lut_i16, tman.tman_mpgemv_i16, tman.tman_mpgemv_i16_batch_run) if integer else
                              (tman.tman_lut_bytes, tman.tman_build_lut, tman.tman_mpgemv, tman.tman_mpgemv_batch_run))
    lut = torch.empty(size(N, shape.K, shape.group), dtype=torch.uint8, device=dev())
    build(to_dev(x), N, shape.K, shape.group, lut)
    ys = [torch.full((N, shape.M), float("nan"), dtype=torch.float16, device=dev()) for _ in range(batch)]
    ws = [gemv_workspace(shape, N) for _ in range(batch)]
    if batch == 1:
        one(shape, blob, lut, N, ys[0], ws[0])
    else:
        desc = torch.empty(tman.tman_mpgemv_batch_desc_bytes(batch), dtype=torch.uint8, device=dev())
        tman.tman_mpgemv_batch_prepare([shape] * batch, [blob] * batch, [lut] * batch, N, ys, ws, desc)
        many([shape] * batch, N, desc)
    torch.cuda.synchronize()
    assert all(torch.equal(y, ys[0]) for y in ys) and torch.isfinite(ys[0]).all()
    row_blocks = -(-shape.M // 64)
    sums = ws[0][-(-row_blocks * 4 // 256) * 256:].cpu().numpy().view(np.float32)
    tokens = 2 if N == 2 else 4 if N <= 4 else 8
    per_segment = tokens * 64
    used = np.flatnonzero(sums)
    if used.size == 0:
        return 1
    segments = -(-(int(used[-1]) + 1) // per_segment) / row_blocks
    assert segments == int(segments)
    return int(segments)


@pytest.fixture
def tiling():
    saved = tman.tman_get_tiling()
    yield lambda **kw: tman.tman_set_tiling(_with(**kw))
    tman.tman_set_tiling(saved)


def _with(**kw):
    t = tman.tman_default_tiling()
    for k, v in kw.items():
        setattr(t, k, v)
    return t


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("bits,N,name", [(4, 2, "decode_seg_tiles"), (4, 4, "decode_seg_tiles_many"), (2, 2, "decode_seg_tiles"),
                                         (2, 8, "decode_seg_tiles_many"), (1, 2, "decode_seg_tiles"), (1, 6, "decode_seg_tiles_many")])
def test_segments_as_the_caller_sets_them(tiling, bits, N, name, integer):
    shape = tman.Shape(64, 40 * 128, bits, 128)
    for tiles, segments in [(10, 4), (20, 2), (64, 1)]:
        tiling(**{name: tiles})
        assert _segments(shape, N, integer) == segments
        assert _segments(shape, N, integer, batch=9) == segments


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("bits,N", [(4, 2), (4, 4), (4, 8), (2, 2), (2, 4), (1, 8)])
def test_short_segments_where_units_are_idle(bits, N, integer):
    """86 tiles: 3 (two tokens) or 4 segments while the launch has no more workgroups than the chip has units, then 2."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    short = 3 if N == 2 else 4
    shape = tman.Shape(64, 86 * 128, bits, 128)
    assert _segments(shape, N, integer) == short
    assert _segments(shape, N, integer, batch=9) == short
    rows = units // short * 64
    assert _segments(tman.Shape(rows, 86 * 128, bits, 128), N, integer) == short
    assert _segments(tman.Shape(rows + 64, 86 * 128, bits, 128), N, integer) == 2
