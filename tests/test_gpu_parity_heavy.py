"""GPU: parities of rows of 32 to 127 words against generators heavier than the
support list, few of them to 64 generators (their bit rows are walked by the
whole wave), many, and around the line between."""
import numpy as np
import pytest
import torch

from paper_2501_04776_amd import api, packing
from tests.test_gpu_parity_rows import _bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [31, 32, 63, 64, 65, 127])
@pytest.mark.parametrize("heavy", [1, 3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 64])  # of every 64 generators
def test_parity_heavy_generators(words, heavy):
    R, C = 200, 300
    n = 64 * words - 3
    rng = np.random.default_rng(100 * words + heavy)
    rows = rng.integers(0, 2, size=(R, n), dtype=np.uint8)
    cols = np.zeros((C, n), dtype=np.uint8)
    for j in range(C):
        w = (9, 11, 200, n)[(j // 7) % 4] if j * 37 % 64 < heavy else j % 9
        cols[j, rng.choice(n, size=w, replace=False)] = 1
    ref = (rows.astype(np.float32) @ cols.T.astype(np.float32)).astype(np.int64) % 2
    dr = torch.from_numpy(packing.pack_dense(rows).view(np.int64)).cuda()
    dc = torch.from_numpy(packing.pack_dense(cols).view(np.int64)).cuda()
    got = api.iqp_parity(dr, dc, n, api.ROW_MAJOR).cpu().numpy().view(np.uint64)
    assert np.array_equal(_bits(got, C), ref)
    Cw, Rw = (C + 63) // 64, (R + 63) // 64
    t = api.iqp_parity(dr, dc, n, api.TILED32).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Cw, 32).transpose(0, 2, 1).reshape(-1, Cw)
    assert np.array_equal(_bits(t[:R], C), ref)
    t = api.iqp_parity(dr, dc, n, api.TILED32_T).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Rw, 32).transpose(0, 2, 1).reshape(-1, Rw)
    assert np.array_equal(_bits(t[:C], R), ref.T)
