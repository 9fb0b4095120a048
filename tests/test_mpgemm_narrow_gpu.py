"""The narrow tiles of the prefill kernel whose waves split K (64 rows x 64 tokens with four or eight waves, 64 x 128),
which the launcher picks by the grid: ragged rows and tokens, K that is no whole number of rounds of the waves."""
import numpy as np
import pytest

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import TOL, mpgemm, pack, rand_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,bits,group,hz,N", [
    (130, 1056, 4, 32, True, 33),     # 64 x 64, four waves: 16.5 stages of 64 columns
    (64, 1024, 2, 64, True, 64),      # ... exactly one token tile, one round
    (65, 2976, 1, 32, False, 129),    # ... three token tiles, the last with one token
    (100, 1088, 1, 64, True, 40),
    (130, 4128, 4, 32, True, 40),     # ... 64.5 stages
    (64, 3072, 2, 128, True, 190),
    (65, 11008, 4, 128, True, 65),    # 64 x 64, eight waves (K from 8192 on): 172 stages
    (8256, 1056, 4, 32, True, 97),    # 64 x 128: 129 row blocks
    (8250, 1152, 2, 128, True, 128),
    (16400, 1024, 1, 64, False, 50),  # 257 workgroups of 64 x 64: a second one on a unit
])
def test_narrow_tiles(oracle_lib, M, K, bits, group, hz, N):
    q, s, z, x = rand_case(4100 + M + K + bits + N, M, K, N, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    assert tman.tman_mpgemm_splits_k(shape, N) == 1 and tman.tman_mpgemm_tile_rows(shape, N) == 64
    y = mpgemm(shape, pack(shape, q, s, z), x)
    assert np.all(np.isfinite(y.astype(np.float32)))
    rows = np.arange(N) if M < 1000 else np.unique([0, 31, 32, 63, 64, N - 2, N - 1])
    rows = rows[rows < N]
    assert oracle.row_relative_error(y[rows], oracle.matmul(q, s, z, x[rows], bits, group)).max() <= TOL
    # the other tokens: the tiled kernel forms the same products, its sums differ in order only (fp32, then one rounding)
    t = tman.tman_get_tiling()
    try:
        tiled = tman.tman_get_tiling()
        tiled.prefill_row_blocks = 2
        tman.tman_set_tiling(tiled)
        assert tman.tman_mpgemm_splits_k(shape, N) == 0
        other = mpgemm(shape, pack(shape, q, s, z), x).astype(np.float64)
    finally:
        tman.tman_set_tiling(t)
    rms = np.sqrt(np.mean(other ** 2, axis=1, keepdims=True))
    assert np.all(np.abs(y - other) <= 2.0 ** -10 * np.maximum(np.abs(other), rms))
