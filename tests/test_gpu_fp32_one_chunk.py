"""GPU: FP32 forwards of 2^31 terms and more with one chunk of samples per
observable (s <= 1024), where the kernels that have the sums write the results
themselves: every observable's phases against the sum they stand for, with more
observables than blocks that run at once, and sums that read as no entry at all."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import _lib as L
from paper_2501_04776_amd import api
from tests.gpu_util import TOL, DevWorkload, grad_tol
from tests.test_gpu_fp32_chain import _phases

pytestmark = pytest.mark.gpu


def _expval(dw):
    """iqp_expval in FP32 into outputs that hold NaN before the call."""
    l, s = dw.ops.shape[0], dw.samples.shape[0]
    mean, se = (torch.full((l,), np.nan, dtype=torch.float64, device="cuda") for _ in range(2))
    ph = torch.full((l, s), np.nan, dtype=torch.float32, device="cuda")
    c = api.Circuit(dw.n, dw.gens, dw.theta).struct()
    nb = api.workspace_bytes(L.IQP_CALL_EXPVAL, dw.n, dw.gens.shape[0], l, s, 0, "fp32")
    ws = torch.full((nb,), 255, dtype=torch.uint8, device="cuda")
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (dw.ops, dw.samples, mean, se, ph, ws)]
    st = L.lib().iqp_expval(ctypes.byref(c), l, ptr[0], s, ptr[1], L.IQP_FP32, *ptr[2:], nb,
                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == L.IQP_OK, L.last_error()
    return mean.cpu().numpy(), se.cpu().numpy(), ph.cpu().numpy()


def _sparse(s, seed, with_data=0):
    # C about 0.6 % full; observable 0, whose block ends first, has weight 0
    w = W.small_random(seed, 400, 1000, 4000, s, gate_w=(1, 2), op_w=(1, 2), with_data=with_data)
    assert w.l * w.s * w.m >= 2 ** 31
    dw = DevWorkload(w)
    dw.ops[0] = 0
    dw.ops01[0] = 0
    return w, dw


@pytest.mark.parametrize("s", [700, 1023, 1024])
def test_fp32_one_chunk_all_rows(s):
    w, dw = _sparse(s, 1200 + s)
    mean, se, ph = _expval(dw)
    ref = _phases(w, dw.ops01, np.arange(w.l), 1)
    # the last FP64 steps may round differently: one FP32 ulp of the phase
    assert (np.abs(ph - ref) <= np.spacing(np.abs(ph))).all()
    assert (ph == ref.astype(np.float32)).mean() > 0.999
    c = np.cos(ph.astype(np.float64))
    # cosf's own rounding, averaged
    assert np.abs(mean - c.mean(axis=1)).max() < 1e-7
    assert np.abs(se - c.std(axis=1) / np.sqrt(s)).max() < 1e-7
    assert mean[0] == 1.0


def test_fp32_one_chunk_gradient_recomputes_the_same_phases():
    w, dw = _sparse(1024, 1300)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    _, _, ph = _expval(dw)
    u = torch.from_numpy(np.random.default_rng(4).normal(size=w.l)).cuda()
    saved = api.iqp_expval_grad(circ, dw.ops, dw.samples, u, torch.from_numpy(ph).cuda(), "fp32")
    assert torch.equal(api.iqp_expval_grad(circ, dw.ops, dw.samples, u, None, "fp32"), saved)


def test_fp32_one_chunk_mmd():
    w, dw = _sparse(700, 1400, with_data=100)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    loss, g = api.iqp_mmd_loss_grad(circ, dw.ops, dw.op_weight, dw.samples, dw.data, True, True,
                                    "fp32")
    ol, og = oracle.mmd_loss_grad(w.n, w.gates, w.theta, dw.ops01, w.op_weight, w.samples, w.data,
                                  True)
    assert abs(loss.item() - ol) < TOL["fp32"]
    assert np.abs(g.cpu().numpy() - og).max() < grad_tol("fp32", og)


def test_fp32_one_chunk_dense_zero_sum():
    # observable 0 anticommutes with two gates of angle pi / 4 alone: its phases
    # are 0 or +-pi and its cosines, over balanced samples, add to exactly 0.
    # The others are on the other qubits: C is dense, the matrix cores' case
    n, m, l, s = 40, 1000, 2200, 1000
    assert l * s * m >= 2 ** 31
    rng = np.random.default_rng(17)
    gates01 = (rng.random((m, n)) < 0.3).astype(np.uint8)
    gates01[:, 0] = 0
    gates01[0] = gates01[1] = 0
    gates01[0, 0] = gates01[1, 0] = gates01[1, 1] = 1
    ops01 = (rng.random((l, n)) < 0.3).astype(np.uint8)
    ops01[:, 0] = 0
    ops01[0] = 0
    ops01[0, 0] = 1
    theta = rng.uniform(-np.pi, np.pi, size=m)
    theta[:2] = np.pi / 4
    z = (rng.random((s, n)) < 0.5).astype(np.uint8)
    z[:, 1] = np.arange(s) % 2
    w = W.Workload("zero sum", n, W.dense_to_rows(gates01), theta, W.dense_to_rows(ops01), z)
    assert oracle.parity(n, ops01, w.gates).mean() > 0.45
    mean, se, _ = _expval(DevWorkload(w))
    om, ose = oracle.expval(n, w.gates, theta, ops01, z)
    assert mean[0] == 0.0
    assert np.abs(mean - om).max() < TOL["fp32"]
    assert np.abs(se - ose).max() < TOL["fp32"]
