"""GPU: parities of rows of 64 to 127 words, from bit columns in LDS and, from 1024
waves of 64 generators and 64 row words on, in memory: every layout on both sides of
the line, the calls built on them, circuits of a batch on different sides, and the
MMD forward that leaves out operators of weight 0."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import BatchPlan, api
from tests.gpu_util import TOL, DevWorkload
from tests.test_gpu_parity_rows import _bits

pytestmark = pytest.mark.gpu


def _rows(rng, r, n, words, weights):
    """r packed rows of about the given weights in turn."""
    x = np.zeros((r, words), dtype=np.uint64)
    wt = np.resize(weights, r)
    for k in range(max(weights)):
        j = np.nonzero(wt > k)[0]
        q = rng.integers(0, n, size=j.size)
        x[j, q // 64] |= np.uint64(1) << (q % 64).astype(np.uint64)
    return x


@pytest.mark.parametrize("words", [63, 64, 127, 128])
@pytest.mark.parametrize("rows,cols", [(70, 65400), (70, 65500), (4200, 32760)])
def test_parity_layouts(words, rows, cols):
    n = 64 * words - 5
    rng = np.random.default_rng(words + rows + cols)
    a = _rows(rng, rows, n, words, (1, 3, 40, 500))
    b = _rows(rng, cols, n, words, (1, 2, 3, 8, 9, 0, 30))
    pick = np.unique(np.r_[0, cols - 1, rng.integers(0, cols, 200)])
    ref = (_bits(a, n).astype(np.float32) @ _bits(b[pick], n).T.astype(np.float32)).astype(
        np.int64) % 2
    da = torch.from_numpy(a.view(np.int64)).cuda()
    db = torch.from_numpy(b.view(np.int64)).cuda()
    Cw, Rw = (cols + 63) // 64, (rows + 63) // 64
    got = api.iqp_parity(da, db, n, api.ROW_MAJOR).cpu().numpy().view(np.uint64)
    assert np.array_equal(_bits(got, cols)[:, pick], ref)
    t = api.iqp_parity(da, db, n, api.TILED32).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Cw, 32).transpose(0, 2, 1).reshape(-1, Cw)
    assert np.array_equal(_bits(t[:rows], cols)[:, pick], ref)
    t = api.iqp_parity(da, db, n, api.TILED32_T).cpu().numpy().view(np.uint64)
    t = t.reshape(-1, Rw, 32).transpose(0, 2, 1).reshape(-1, Rw)
    assert np.array_equal(_bits(t[pick], rows), ref.T)


@pytest.mark.parametrize("prec", ["sparse_fp32", "fp32", "split_bf16"])
def test_calls_match_more_words(prec):
    """The same circuit at 65 words (columns from 1024 waves on) and 33 (LDS)."""
    n, m, l, s = 2100, 65500, 40, 1200
    w = W.small_random(5, n, m, l, s, theta_scale=0.1)
    dw = DevWorkload(w)
    u = torch.from_numpy(np.random.default_rng(6).normal(size=l)).cuda()

    def wide(x):
        return torch.cat([x, torch.zeros((x.shape[0], 65 - x.shape[1]), dtype=x.dtype,
                                         device=x.device)], 1).contiguous()

    res = []
    for f, q in ((lambda x: x, n), (wide, 64 * 65)):
        circ = api.Circuit(q, f(dw.gens), dw.theta)
        mean, se, ph = api.iqp_expval(circ, f(dw.ops), f(dw.samples), prec, phase_save=True)
        g = api.iqp_expval_grad(circ, f(dw.ops), f(dw.samples), u, ph, prec)
        res.append((mean, se, ph, g))
    for x, y in zip(*res):  # the parities are bits, all else runs alike
        assert torch.equal(x, y)


def test_batch_of_both_forms():
    us, plan_in, single = [], [], []
    for i, (n, m, l, s) in enumerate([(4100, 40000, 70, 300), (4100, 300, 90, 200),
                                      (300, 2000, 50, 400), (8200, 500, 30, 100)]):
        w = W.small_random(60 + i, n, m, l, s, theta_scale=0.1)
        dw = DevWorkload(w)
        us.append(torch.from_numpy(np.random.default_rng(i).normal(size=l)).cuda())
        plan_in.append((api.Circuit(n, dw.gens, dw.theta), dw.ops, dw.samples))
        mean, _, ph = api.iqp_expval(*plan_in[-1], "split3_bf16", phase_save=True)
        single.append((mean, api.iqp_expval_grad(*plan_in[-1], us[-1], ph, "split3_bf16")))
    plan = BatchPlan(plan_in, "split3_bf16")
    means, _ = plan.expval()
    grads = plan.expval_grad(us)
    for i, (mean, g) in enumerate(single):
        # FP32 partial sums may be split differently
        assert float((means[i] - mean).abs().max()) < TOL["split3_bf16"] / 10
        assert float((grads[i] - g).abs().max()) < TOL["split3_bf16"] / 10 * max(
            1.0, float(g.abs().max()))
    plan.close()


def test_mmd_without_weight_zero():
    n, m, l, s = 4100, 66000, 240, 1100
    w = W.small_random(8, n, m, l, s, theta_scale=0.1, with_data=30)
    ops = W.rows_to_dense(w.ops, n)
    rng = np.random.default_rng(9)
    ops[rng.random(l) < 0.5] = 0
    w.ops = W.dense_to_rows(ops)
    assert l * s * m >= 2 ** 34
    dw = DevWorkload(w)
    circ = api.Circuit(n, dw.gens, dw.theta)
    wt = torch.from_numpy(rng.random(l)).cuda()
    a = api.iqp_mmd_loss_grad(circ, dw.ops, wt, dw.samples, dw.data, True, True, "split3_bf16")
    b = api.iqp_mmd_loss_grad(circ, dw.ops, wt, dw.samples, dw.data, True, True, "sparse_fp32")
    scale = max(1.0, float(wt.sum()))
    assert abs(a[0].item() - b[0].item()) < TOL["split3_bf16"] * scale
    assert float((a[1] - b[1]).abs().max()) < TOL["split3_bf16"] * max(
        1.0, float(b[1].abs().max()))
