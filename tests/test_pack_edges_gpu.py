"""Packing at the edges of its workgroups: several K tiles per workgroup, rows and columns beyond the matrix, codes that
are not 16-byte aligned (read byte by byte) and codes with bits above the format's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_11248_amd as tman
from gpu_helpers import dev, rand_case, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,hz", [(1, True), (1, False), (2, True), (4, True)])
@pytest.mark.parametrize("M,K,group", [(1, 32, 32), (65, 128, 128), (130, 1088, 64), (9000, 2080, 32), (64, 8320, 64)])
@pytest.mark.parametrize("offset", [0, 1, 8])
def test_blob_is_the_reference_blob(oracle_lib, M, K, group, bits, hz, offset):
    q, s, z, _ = rand_case(M + K + bits, M, K, 1, bits, group, hz)
    shape = tman.Shape(M, K, bits, group, hz)
    raw = torch.zeros(M * K + 16, dtype=torch.uint8, device=dev())
    codes = raw[offset:offset + M * K]
    codes.copy_(to_dev(q.reshape(-1) | np.uint8(0xF0 if bits == 4 else 0xA0)))  # the packer ignores the upper bits
    blob = torch.full((tman.tman_packed_bytes(shape),), 0xA5, dtype=torch.uint8, device=dev())
    tman.tman_pack_weights(shape, codes, to_dev(s), to_dev(z), blob)
    torch.cuda.synchronize()
    assert np.array_equal(blob.cpu().numpy(), oracle.pack_reference(q, s, z, bits, group))
