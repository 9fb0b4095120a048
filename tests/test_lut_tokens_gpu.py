"""Table builders with several threads per table: every padded token count, K below and above what a block's threads search in
one step, activations at every alignment."""
import math

import numpy as np
import pytest
import torch

import paper_2511_11248_amd as tman
import synth
from gpu_helpers import dev

pytestmark = pytest.mark.gpu


def _build(integer, x, group):
    N, K = x.shape
    size, build = (tman.tman_lut_i16_bytes, tman.tman_build_lut_i16) if integer else (tman.tman_lut_bytes, tman.tman_build_lut)
    lut = torch.zeros(size(N, K, group), dtype=torch.uint8, device=dev())
    build(x, N, K, group, lut)
    torch.cuda.synchronize()
    return lut


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("K,group", [(32, 32), (192, 64), (8224, 32), (12416, 128)])
def test_alignment_of_the_activations(K, group, N, integer):
    host = torch.from_numpy(synth.normal_fp16(900 + K + N, N * K))
    tables = []
    for offset in (0, 4, 1):  # 16, 8 and 2 bytes
        room = torch.empty(N * K + 8, dtype=torch.float16, device=dev())
        x = room[offset:offset + N * K]
        x.copy_(host)
        assert x.data_ptr() % 16 == 2 * offset
        tables.append(_build(integer, x.view(N, K), group))
    assert torch.equal(tables[0], tables[1]) and torch.equal(tables[0], tables[2])


@pytest.mark.parametrize("N", [1, 2, 5])
@pytest.mark.parametrize("K,at", [(96, 95), (8224, 6150), (12416, 12415)])
def test_integer_entries(K, at, N):
    """The largest magnitude anywhere in the row sets the step; entries and block sums are exact integers."""
    group = 32
    x = synth.normal_fp16(950 + K, N * K).reshape(N, K)
    x[:, at] = [30.0 * (n + 1) for n in range(N)]
    lut = _build(True, torch.from_numpy(x).to(dev()), group).cpu().numpy()
    NP = 1 if N == 1 else 2 if N == 2 else 8
    nkt = -(-K // 128)
    entries = lut[:nkt * 1024 * NP].view(np.int16).reshape(nkt * 32, 16, NP)
    sums = lut[nkt * 1024 * NP:nkt * 1024 * NP + nkt * 4 * NP * 4].view(np.int32).reshape(nkt * 4, NP)
    for n in range(N):
        e = math.frexp(float(np.abs(x[n].astype(np.float64)).max()))[1] - 13
        xq = np.zeros(nkt * 128, dtype=np.int64)
        xq[:K] = np.rint(x[n].astype(np.float64) * 2.0 ** -e)
        want = np.stack([sum(xq.reshape(-1, 4)[:, t] * (p >> t & 1) for t in range(4)) for p in range(16)], axis=1)
        assert np.array_equal(entries[:, :, n], want)
        assert np.array_equal(sums[:, n], xq.reshape(-1, 32).sum(axis=1))
    assert not entries[:, :, N:].any() and not sums[:, N:].any()
