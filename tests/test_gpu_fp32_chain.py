"""GPU: the FP32 forward over the non-zero entries of C against the sum it
stands for, bit by bit: per gate split the running FP32 sum of +-2 theta'_j
over the anticommuting gates in gate order, the splits added in FP64 and
reduced modulo 2 pi. Sizes around the lane, wave, block and list limits, on
both sides of the density rule (above it the matrix cores give the same sum)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload, check_grad

pytestmark = pytest.mark.gpu

TWO_PI_HI, TWO_PI_LO = 6.283185307179586, 2.4492935982947064e-16


def _phases(w, ops01, rows, splits):
    """Phases of the observables `rows` in the arithmetic of the FP32 form."""
    th = w.theta - np.pi * np.rint(w.theta * 0.3183098861837907)
    t = (2.0 * th).astype(np.float32)
    mw = (w.m + 127) // 128 * 2
    wps = -(-mw // splits)
    C = oracle.parity(w.n, ops01[rows], w.gates)
    B = oracle.parity(w.n, w.samples, w.gates)
    out = np.empty((len(rows), w.s))
    for x, _ in enumerate(rows):
        E = np.zeros(w.s)
        J = np.nonzero(C[x])[0]
        for sp in range(splits):
            acc = np.zeros(w.s, dtype=np.float32)
            for j in J[(J // 64 >= sp * wps) & (J // 64 < (sp + 1) * wps)]:
                acc = acc + np.where(B[:, j] != 0, -t[j], t[j]).astype(np.float32)
            E += acc.astype(np.float64)
        k = np.rint(E * 0.15915494309189535)
        out[x] = (E - k * TWO_PI_HI) - k * TWO_PI_LO
    return out


# (n, m, l, s, gate weight, op weight, splits)
@pytest.mark.parametrize("shape", [
    (400, 5000, 400, 1301, (1, 2), (1, 2), 1),    # C about 1 % full: non-zero entries
    (400, 5000, 400, 2048, (1, 2), (1, 2), 3),    # the same, three gate splits
    (300, 5000, 211, 2057, (1, 3), (1, 3), 2),    # one sample past a block, odd rows
    (90, 30000, 40, 1799, (1, 2), (1, 4), 1),     # rows longer than one list fill
    (40, 5000, 400, 1301, (4, 4), (8, 8), 1),  # C 43 % full: matrix cores
])
def test_fp32_phases_bitwise(shape, monkeypatch):
    n, m, l, s, gw, ow, splits = shape
    assert l * s * m >= 2 ** 31
    monkeypatch.setenv("IQP_FWD_SPLITS", str(splits))
    w = W.small_random(n + m + l + s, n, m, l, s, gate_w=gw, op_w=ow)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    mean, se, ph = api.iqp_expval(circ, dw.ops, dw.samples, "fp32", phase_save=True)
    rows = [0, 1, l // 2, l - 1]
    got = ph.cpu().numpy()[rows]
    ref = _phases(w, dw.ops01, rows, splits)
    # the last FP64 steps may round differently: one FP32 ulp of the phase
    assert (np.abs(got - ref) <= np.spacing(np.abs(got).astype(np.float32))).all()
    assert (got == ref.astype(np.float32)).mean() > 0.999
    c = np.cos(ph.cpu().numpy().astype(np.float64))
    # cosf's own rounding, averaged
    assert np.abs(mean.cpu().numpy() - c.mean(axis=1)).max() < 1e-7
    assert np.abs(se.cpu().numpy() - c.std(axis=1) / np.sqrt(s)).max() < 1e-7


def test_fp32_nan_and_identity_rows():
    # a NaN angle reaches the observables that anticommute with its gate only
    w = W.small_random(77, 400, 5000, 400, 1301, gate_w=(1, 2), op_w=(1, 2))
    w.theta[1234] = np.nan
    dw = DevWorkload(w)
    dw.ops[7] = 0
    ops01 = dw.ops01.copy()
    ops01[7] = 0
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    mean, _, _ = api.iqp_expval(circ, dw.ops, dw.samples, "fp32")
    hit = oracle.parity(w.n, ops01, w.gates)[:, 1234] != 0
    got = mean.cpu().numpy()
    assert hit.any() and np.array_equal(np.isnan(got), hit)
    assert got[7] == 1.0


# (n, m, l, s, gate weight, op weight): C below the density limit, rows of
# less and more than one list fill, ragged samples, one and several blocks of
# 64 observables
@pytest.mark.parametrize("shape", [
    (400, 5000, 400, 1301, (1, 2), (1, 2)),
    (300, 9000, 129, 2057, (1, 3), (1, 3)),
    (90, 30000, 40, 1799, (1, 2), (1, 4)),
    (500, 60000, 17, 2112, (1, 4), (1, 9)),
])
def test_fp32_gradient_bitwise(shape, monkeypatch):
    # the batched form always takes the matrix cores, over one sample split
    n, m, l, s, gw, ow = shape
    assert l * s * m >= 2 ** 31
    monkeypatch.setenv("IQP_BWD_SPLITS", "1")
    w = W.small_random(n + m + l + s, n, m, l, s, gate_w=gw, op_w=ow)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, "fp32", phase_save=True)
    u = torch.from_numpy(np.random.default_rng(8).normal(size=l)).cuda()
    u[l // 3] = 0.0
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, u, ph, "fp32")
    plan = api.BatchPlan([(circ, dw.ops, dw.samples)], "fp32")
    plan.phases[0].copy_(ph)
    (ref,) = plan.expval_grad([u])
    assert torch.equal(g, ref)


@pytest.mark.parametrize("splits", [2, 5, 8, 9])
def test_fp32_gradient_splits(splits, monkeypatch):
    monkeypatch.setenv("IQP_BWD_SPLITS", str(splits))
    w = W.small_random(3100 + splits, 400, 5000, 400, 1301, gate_w=(1, 2), op_w=(1, 2))
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    u = np.random.default_rng(9).normal(size=w.l)
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, torch.from_numpy(u).cuda(), None, "fp32")
    check_grad("fp32", g.cpu().numpy(), w, dw.ops01, u)


def test_fp32_gradient_nan_weight():
    # a NaN weight reaches the gates of its observable only
    w = W.small_random(91, 400, 5000, 400, 1301, gate_w=(1, 2), op_w=(1, 2))
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    u = np.random.default_rng(9).normal(size=w.l)
    u[5] = np.nan
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, torch.from_numpy(u).cuda(), None, "fp32")
    hit = oracle.parity(w.n, dw.ops01[5:6], w.gates)[0] != 0
    assert hit.any() and np.array_equal(np.isnan(g.cpu().numpy()), hit)
