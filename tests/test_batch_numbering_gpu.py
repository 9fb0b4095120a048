"""Table batches whose workgroups are numbered for balance against the same batches on the plain grid: the numbering says
which compute unit runs which workgroup, the outputs are the same bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import TOL, dev, gemv_workspace, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu

DIMS = [(700, 4224), (64, 4224), (1300, 1024), (130, 1024)]  # (M, K): segments of several lengths, ragged row blocks


@pytest.fixture
def balance():
    """Sets tiling.decode_balance: 1 numbers a batch that fits the chip (this one does), 0 is the plain grid."""
    saved = tman.tman_get_tiling()

    def set_to(value):
        t = tman.tman_get_tiling()
        t.decode_balance = value
        tman.tman_set_tiling(t)

    yield set_to
    tman.tman_set_tiling(saved)


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("bits,group,N", [(4, 128, 2), (4, 32, 8), (4, 64, 4), (2, 64, 3), (1, 32, 8)])
def test_numbered_and_plain_table_batches(oracle_lib, balance, bits, group, N, integer):
    shapes, blobs, luts, wss, ys, refs, xs = [], [], {}, [], [], [], {}
    lut_bytes, build, run = ((tman.tman_lut_i16_bytes, tman.tman_build_lut_i16, tman.tman_mpgemv_i16_batch_run) if integer
                             else (tman.tman_lut_bytes, tman.tman_build_lut, tman.tman_mpgemv_batch_run))
    for i, (M, K) in enumerate(DIMS):
        q, s, z, x = rand_case(8200 + i + bits, M, K, N, bits, group)
        shape = tman.Shape(M, K, bits, group)
        if K not in luts:
            xs[K] = x
            luts[K] = torch.empty(lut_bytes(N, K, group), dtype=torch.uint8, device=dev())
            build(to_dev(x), N, K, group, luts[K])
        shapes.append(shape)
        blobs.append(pack(shape, q, s, z))
        wss.append(gemv_workspace(shape, N))
        ys.append(torch.empty((N, M), dtype=torch.float16, device=dev()))
        refs.append(oracle.matmul(q, s, z, xs[K], bits, group))
    desc = torch.empty(tman.tman_mpgemv_batch_desc_bytes(len(shapes)), dtype=torch.uint8, device=dev())
    out = []
    for value in (1, 0):
        balance(value)
        for y in ys:
            y.fill_(float("nan"))
        tman.tman_mpgemv_batch_prepare(shapes, blobs, [luts[s.K] for s in shapes], N, ys, wss, desc)
        for _ in range(2):  # the second pass finds the tickets the first one left
            run(shapes, N, desc)
        torch.cuda.synchronize()
        out.append([y.cpu().numpy() for y in ys])
    for a, b, ref in zip(*out, refs):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
        assert oracle.row_relative_error(a, ref).max() <= TOL
