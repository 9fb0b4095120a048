"""Outputs at addresses that no vector store may assume: y one, four and eight elements into a buffer (2, 8 and 16 bytes), rows of a
multiple of 8 elements.  The same bits as at the buffer's start, and nothing written beside them."""
import numpy as np
import pytest
import torch

import paper_2511_11248_amd as tman
from gpu_helpers import dev, gemv_workspace, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu

M, K, GROUP = 136, 5632, 64  # a ragged row block, two segments


def _at_every_offset(n, run):
    first = None
    for offset in (0, 1, 4, 8):
        room = torch.full((n + 24,), 777.0, dtype=torch.float16, device=dev())
        run(room[8 + offset:8 + offset + n])
        torch.cuda.synchronize()
        got = room.cpu().numpy().view(np.uint16)
        mark = np.float16(777.0).view(np.uint16)
        assert np.all(got[:8 + offset] == mark) and np.all(got[8 + offset + n:] == mark)
        y = got[8 + offset:8 + offset + n]
        first = y if first is None else first
        assert np.array_equal(y, first)
    assert np.isfinite(first.view(np.float16)).all()


def _case(N, bits, group=GROUP, seed=0):
    q, s, z, x = rand_case(11000 + N + bits + seed, M, K, N, bits, group)
    shape = tman.Shape(M, K, bits, group)
    return shape, pack(shape, q, s, z), to_dev(x)


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("N,bits", [(1, 4), (1, 2), (2, 1), (2, 2), (2, 4), (4, 1), (5, 4), (8, 1), (8, 2)])
def test_tables(N, bits, integer):
    shape, blob, x = _case(N, bits)
    size, build, one, many = ((tman.tman_lut_i16_bytes, tman.tman_build_lut_i16, tman.tman_mpgemv_i16, tman.tman_mpgemv_i16_batch_run) if integer else
                              (tman.tman_lut_bytes, tman.tman_build_lut, tman.tman_mpgemv, tman.tman_mpgemv_batch_run))
    lut = torch.empty(size(N, K, GROUP), dtype=torch.uint8, device=dev())
    build(x, N, K, GROUP, lut)
    _at_every_offset(N * M, lambda y: one(shape, blob, lut, N, y, gemv_workspace(shape, N)))

    def batch(y):
        other = torch.empty(N * M, dtype=torch.float16, device=dev())
        desc = torch.empty(tman.tman_mpgemv_batch_desc_bytes(2), dtype=torch.uint8, device=dev())
        ws = [gemv_workspace(shape, N), gemv_workspace(shape, N)]
        tman.tman_mpgemv_batch_prepare([shape] * 2, [blob] * 2, [lut] * 2, N, [other, y], ws, desc)
        many([shape] * 2, N, desc)
        torch.cuda.synchronize()

    _at_every_offset(N * M, batch)


@pytest.mark.parametrize("N,group", [(1, 64), (8, 32), (16, 64), (20, 64), (32, 128), (40, 64), (130, 64), (600, 64)])
def test_mpgemm(N, group):
    shape, blob, x = _case(N, 4, group)

    def run(y):
        need = tman.tman_mpgemm_workspace_bytes(shape, N)
        tman.tman_mpgemm(shape, blob, x, N, y, torch.zeros(need, dtype=torch.uint8, device=dev()) if need else None)

    _at_every_offset(N * M, run)


@pytest.mark.parametrize("k_split", [1, 2, 3])
def test_mpgemm_prefill_kernels(k_split):
    saved = tman.tman_get_tiling()
    t = tman.tman_get_tiling()
    t.prefill_k_split = k_split
    tman.tman_set_tiling(t)
    try:
        test_mpgemm(70, 64)
    finally:
        tman.tman_set_tiling(saved)


@pytest.mark.parametrize("blocks", [1, 3, 9])
def test_mpgemm_i8(blocks):
    N = 70
    shape, blob, x = _case(N, 2, seed=1)
    xq = torch.empty(tman.tman_act_i8_bytes(N, K), dtype=torch.uint8, device=dev())
    tman.tman_quantize_act_i8(x, N, K, xq)
    saved = tman.tman_get_tiling()
    t = tman.tman_get_tiling()
    t.i8_token_blocks = blocks
    tman.tman_set_tiling(t)
    try:
        _at_every_offset(N * M, lambda y: tman.tman_mpgemm_i8(shape, blob, xq, N, y))
    finally:
        tman.tman_set_tiling(saved)
