"""One-token decode (4-bit weights and integer tables: the 4-bit dot product unit; 1- and 2-bit weights: the matrix cores): precision,
infinities and NaN, agreement of its three sources of activations (x, fp16 tables, int16 tables)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import dev, gemv_workspace, mpgemv, mpgemv_x, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu

FORMATS = [(1, True), (1, False), (2, True), (4, True)]
EDGES = [(65, 128), (40, 160), (64, 2048), (33, 2080), (70, 4096), (64, 4224)]  # passes, last tile, two segments


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("M,K", EDGES)
def test_short_activations_are_not_rounded(oracle_lib, M, K, group, bits, hz):
    """Activations that are 10-bit integers times a power of two per block enter the sums exactly (as 16-bit integers; as digits, which
    hold 17 bits below a block's largest), so the only roundings are the fp32 sum over blocks and the fp16 result: half a step of the result, 2^-11, plus the fp32 terms
    (K / group additions of 2^-24 each, against the largest partial sum, taken as 64 times the row's rms)."""
    K = -(-K // group) * group
    q, s, z, _ = rand_case(500 + M + K + bits + group, M, K, 1, bits, group, hz)
    rng = np.random.default_rng(M * K + bits)
    e = rng.integers(-8, 5, size=K // group).repeat(group)
    x = (rng.integers(-1023, 1024, size=K) * np.exp2(e - 10.0)).astype(np.float16).reshape(1, K)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    Y = oracle.matmul(q, s, z, x, bits, group)
    bound = 2.0 ** -11 * np.maximum(np.abs(Y), 2.0 ** -14) + 64 * (K // group) * 2.0 ** -24 * np.sqrt(np.mean(Y ** 2))
    for y in (mpgemv_x(shape, blob, x), mpgemv(shape, blob, x)):
        assert np.all(np.abs(y.astype(np.float64) - Y) <= bound)


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("through_tables", [False, True])
def test_infinities_and_nan(oracle_lib, bits, hz, through_tables):
    """Single activations that are infinite or NaN, next to finite ones, as in the sum over all columns: +-inf by the
    sign of the weight, NaN for a NaN, for a zero weight and where infinities of both signs meet."""
    M, K, group = 66, 4352, 64  # two segments
    q, s, z, x = rand_case(900 + bits, M, K, 1, bits, group, hz)
    if z is not None:
        z[:] = np.float16(1.0)  # codes equal to the zero make the product 0 * inf
    w = ((2.0 * q - 1.0) if z is None else q - z.astype(np.float64).repeat(group, axis=1)) * s.astype(np.float64).repeat(group, axis=1)
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    run = mpgemv if through_tables else mpgemv_x
    for place, value in [((0,), np.inf), ((4351,), -np.inf), ((131, 2177), np.inf), ((64, 4200), np.nan)]:
        xi = x.copy()
        xi[0, list(place)] = value
        if value == np.inf and len(place) == 2:
            xi[0, place[1]] = -np.inf
        with np.errstate(invalid="ignore"):
            ref = (w * xi.astype(np.float64)).sum(axis=1)
        y = run(shape, blob, xi)[0].astype(np.float64)
        assert np.array_equal(np.isnan(y), np.isnan(ref))
        assert np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("group,outlier", [(32, 100), (128, 20), (128, 100), (128, 1000)])
def test_outlier_channels(oracle_lib, group, outlier, bits, hz):
    """1 % of the channels 20 to 1000 times the others.  The error is that of the fp16 result (a step of the result,
    uniform: / sqrt(12)) and of activations that are not multiples of their step (a step, uniform, times the weight).  4 bits: a quantization
    block's step is the smallest 2^e with max |x| <= 30583 * 2^e.  1 and 2 bits: 32 columns have the step 2^-18 times the power of two
    above their largest.  Both sums have thousands of terms, so their rms is known to a few per cent."""
    M, K = 1024, 4096
    q, s, z, _ = rand_case(820 + bits + group, M, K, 1, bits, group, hz)
    rng = np.random.default_rng(outlier + group)
    x = rng.standard_normal(K)
    x[rng.permutation(K)[:K // 100]] *= outlier
    x = x.astype(np.float16).reshape(1, K)
    w = ((2.0 * q - 1.0) if z is None else q - z.astype(np.float64).repeat(group, axis=1)) * s.astype(np.float64).repeat(group, axis=1)
    xd = x[0].astype(np.float64)
    Y = w @ xd
    if bits == 4:
        step = np.exp2(np.ceil(np.log2(np.abs(xd).reshape(-1, group).max(axis=1) / 30583.0))).repeat(group)
    else:
        step = np.exp2(np.ceil(np.log2(np.abs(xd).reshape(-1, 32).max(axis=1))) - 18).repeat(32)
    rounded = np.rint(xd / step) != xd / step
    half = np.exp2(np.maximum(np.floor(np.log2(np.abs(Y) + 1e-30)), -14) - 10)
    expected = np.sqrt(np.mean(((w * w) @ np.where(rounded, step * step, 0.0) + half * half) / 12.0))
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    for y in (mpgemv_x(shape, blob, x), mpgemv(shape, blob, x)):
        assert np.sqrt(np.mean((y[0].astype(np.float64) - Y) ** 2)) <= 1.1 * expected


def test_largest_activations_stay_finite(oracle_lib):
    """Four activations of 65504 sum past the largest fp16 number; sums of digits do not overflow."""
    M, K, bits, group = 64, 256, 4, 128
    q, s, z, _ = rand_case(77, M, K, 1, bits, group)
    s[:] = np.float16(2.0 ** -12)
    x = np.full((1, K), 65504.0, dtype=np.float16)
    shape = tman.Shape(M, K, bits, group)
    Y = oracle.matmul(q, s, z, x, bits, group)
    assert np.abs(Y).max() < 65504
    assert oracle.row_relative_error(mpgemv_x(shape, pack(shape, q, s, z), x), Y).max() <= 1e-3


@pytest.mark.parametrize("bits,hz", FORMATS)
@pytest.mark.parametrize("K", [96, 2080, 4224])
def test_sources_agree(oracle_lib, K, bits, hz):
    """x, fp16 tables and int16 tables of the same short activations give the same sums: the results differ by the
    order of the fp32 additions at most, one step of the fp16 result."""
    M, group = 130, 32
    q, s, z, _ = rand_case(40 + K + bits, M, K, 1, bits, group, hz)
    x = np.random.default_rng(K).integers(-2047, 2048, size=(1, K)).astype(np.float16)
    x[0, 0] = 2047  # fixes the int16 step at 1/4
    shape = tman.Shape(M, K, bits, group, hz)
    blob = pack(shape, q, s, z)
    lut = torch.empty(tman.tman_lut_i16_bytes(1, K, group), dtype=torch.uint8, device=dev())
    y16 = torch.empty((1, M), dtype=torch.float16, device=dev())
    tman.tman_build_lut_i16(to_dev(x), 1, K, group, lut)
    tman.tman_mpgemv_i16(shape, blob, lut, 1, y16, gemv_workspace(shape, 1))
    torch.cuda.synchronize()
    a, b, c = (v[0].astype(np.float64) for v in (mpgemv_x(shape, blob, x), mpgemv(shape, blob, x), y16.cpu().numpy()))
    rms = np.sqrt(np.mean(a ** 2))
    assert np.all(np.abs(a - b) <= 2.0 ** -10 * np.maximum(np.abs(a), rms))
    assert np.all(np.abs(a - c) <= 2.0 ** -10 * np.maximum(np.abs(a), rms))
