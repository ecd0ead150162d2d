"""GPU: parities at the row widths where the kernel's blocking changes (row
words per block 16, 8, 4, 2, 1, and the bit-column kernels past them), ragged
row and generator counts, generators heavier than the support list; and the
forward's wave tile rule, which may not change a bit."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import api, packing
from tests.gpu_util import DevWorkload

pytestmark = pytest.mark.gpu


def _bits(words, count):
    return np.unpackbits(words.astype("<u8").view(np.uint8).reshape(words.shape[0], -1), axis=1,
                         bitorder="little")[:, :count]


@pytest.mark.parametrize("words", [1, 7, 8, 17, 18, 31, 32, 63, 64, 127, 128])
@pytest.mark.parametrize("shape", [(1, 1), (130, 65), (1100, 700)])
def test_parity_layouts(words, shape):
    R, C = shape
    n = 64 * words - (3 if words > 1 else 50)
    rng = np.random.default_rng(1000 * words + R)
    rows = rng.integers(0, 2, size=(R, n), dtype=np.uint8)
    cols = np.zeros((C, n), dtype=np.uint8)
    for j in range(C):
        w = [1, 2, 3, 8, min(9, n), min(20, n), 0][j % 7]
        cols[j, rng.choice(n, size=min(w, n), replace=False)] = 1
    ref = (rows.astype(np.float32) @ cols.T.astype(np.float32)).astype(np.int64) % 2
    dr = torch.from_numpy(packing.pack_dense(rows).view(np.int64)).cuda()
    dc = torch.from_numpy(packing.pack_dense(cols).view(np.int64)).cuda()
    got = api.iqp_parity(dr, dc, n, api.ROW_MAJOR).cpu().numpy().view(np.uint64)
    assert np.array_equal(_bits(got, C), ref)
    Cw, Rw = (C + 63) // 64, (R + 63) // 64
    t = api.iqp_parity(dr, dc, n, api.TILED32).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Cw, 32).transpose(0, 2, 1).reshape(-1, Cw)
    assert np.array_equal(_bits(t[:R], C), ref) and not t[R:].any()
    t = api.iqp_parity(dr, dc, n, api.TILED32_T).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Rw, 32).transpose(0, 2, 1).reshape(-1, Rw)
    assert np.array_equal(_bits(t[:C], R), ref.T) and not t[C:].any()


@pytest.mark.parametrize("n", [60, 700, 1100, 2100, 4100, 8300])
def test_sparse_rows_match_dense(n):
    # the sparse form's C and B^T (row-major) against the dense form's bits
    w = W.small_random(n, n, 1500, 70, 1100)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    a, _, _ = api.iqp_expval(circ, dw.ops, dw.samples, "sparse_fp32")
    b, _, _ = api.iqp_expval(circ, dw.ops, dw.samples, "fp32")
    assert float((a - b).abs().max()) < 2e-5  # 1e-5 each against the exact means


@pytest.mark.parametrize("prec", ["fp32", "split_bf16", "split3_bf16"])
@pytest.mark.parametrize("shape", [(10, 55, 100, 1000), (70, 1000, 257, 1025)])
def test_forward_tile_does_not_change_bits(prec, shape, monkeypatch):
    n, m, l, s = shape
    w = W.small_random(7, n, m, l, s)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    mean, se, ph = api.iqp_expval(circ, dw.ops, dw.samples, prec, phase_save=True)
    for tile in ("4x4", "2x4", "2x2"):
        monkeypatch.setenv("IQP_FWD_TILE", tile)
        m2, s2, p2 = api.iqp_expval(circ, dw.ops, dw.samples, prec, phase_save=True)
        assert torch.equal(ph, p2) and torch.equal(mean, m2) and torch.equal(se, s2)
