"""One-token batches of 1-bit weights so large that a workgroup takes two row blocks with one set of digits: the same
bits as single calls, from activations and from tables, at row blocks and rows that do not divide."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import TOL, build_lut, dev, gemv_workspace, pack, rand_case, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("through_tables", [False, True])
@pytest.mark.parametrize("group,hz", [(32, True), (64, False), (128, True)])
def test_two_row_blocks_per_workgroup(oracle_lib, group, hz, through_tables):
    """Nine GEMVs (a batch of more than eight is not numbered); the first makes up the workgroups, more than sixteen per
    compute unit.  Odd and even numbers of row blocks, one and several K segments."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    big = 64 * (16 * units + 3) - 5
    dims = [(big, 128), (130, 4224), (64, 2080), (1, 128), (65, 4096), (257, 384), (320, 160), (192, 8320), (700, 1024)]
    shapes, blobs, xs, ys, wss, cases = [], [], [], [], [], []
    for i, (M, K) in enumerate(dims):
        K = -(-K // group) * group
        q, s, z, x = rand_case(9300 + i + group, M, K, 1, 1, group, hz)
        if i == 2:
            x[0, 70] = np.inf
        shape = tman.Shape(M, K, 1, group, hz)
        shapes.append(shape)
        blobs.append(pack(shape, q, s, z))
        xs.append(build_lut(to_dev(x), group) if through_tables else to_dev(x))
        ys.append(torch.full((1, M), float("nan"), dtype=torch.float16, device=dev()))
        wss.append(gemv_workspace(shape, 1))
        cases.append((q, s, z, x))
    desc = torch.empty(tman.tman_mpgemv_batch_desc_bytes(len(shapes)), dtype=torch.uint8, device=dev())
    if through_tables:
        tman.tman_mpgemv_batch_prepare(shapes, blobs, xs, 1, ys, wss, desc)
    else:
        tman.tman_mpgemv_x_batch_prepare(shapes, blobs, xs, ys, wss, desc)
    for _ in range(2):  # the second pass finds the tickets the first one left
        if through_tables:
            tman.tman_mpgemv_batch_run(shapes, 1, desc)
        else:
            tman.tman_mpgemv_x_batch_run(shapes, desc)
    torch.cuda.synchronize()
    for i, (shape, blob, x, y) in enumerate(zip(shapes, blobs, xs, ys)):
        single = torch.full((1, shape.M), float("nan"), dtype=torch.float16, device=dev())
        if through_tables:
            tman.tman_mpgemv(shape, blob, x, 1, single, gemv_workspace(shape, 1))
        else:
            tman.tman_mpgemv_x(shape, blob, x, single, gemv_workspace(shape, 1))
        torch.cuda.synchronize()
        a, b = y.cpu().numpy(), single.cpu().numpy()
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), dims[i]
        q, s, z, xh = cases[i]
        if i != 2:
            assert oracle.row_relative_error(a, oracle.matmul(q, s, z, xh, 1, group)).max() <= TOL, dims[i]
