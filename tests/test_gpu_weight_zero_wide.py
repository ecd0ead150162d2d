"""GPU: observables of weight 0 among observables whose only qubit is in the first
or the last word of 64, or past the first 64 words, of rows of 1 to 80 words: the
sparse kernels skip exactly the former."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import TOL, DevWorkload, check_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [1, 2, 63, 64, 65, 80])
def test_single_qubit_observables(words):
    n, m, l, s = 64 * words - 1, 600, 12, 1100
    w = W.small_random(40 + words, n, m, l, s, theta_scale=0.3)
    last = 64 * (words - 1)
    qubits = [0, n - 1, last, max(last - 1, 0), min(63, n - 1), min(4096, n - 1)]
    ops = np.zeros((l, n), dtype=np.uint8)
    for i, q in enumerate(qubits):
        ops[2 * i, q] = 1  # the odd ones stay at weight 0
    w.ops = W.dense_to_rows(ops)
    gates = W.rows_to_dense(w.gates, n)
    for i, q in enumerate(qubits):  # none of them commutes with all
        gates[i] = 0
        gates[i, q] = 1
    w.gates = W.dense_to_rows(gates)
    dw = DevWorkload(w)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    u = np.random.default_rng(3).normal(size=l)
    mean, se, ph = api.iqp_expval(circ, dw.ops, dw.samples, "sparse_fp32", phase_save=True)
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, torch.from_numpy(u).cuda(), ph,
                            "sparse_fp32")
    om, _ = oracle.expval(w.n, w.gates, w.theta, dw.ops01, w.samples)
    assert np.abs(mean.cpu().numpy() - om).max() < TOL["sparse_fp32"]
    assert (mean[1::2] == 1.0).all() and (se[1::2] == 0.0).all() and (ph[1::2] == 0.0).all()
    assert (ph[0::2] != 0.0).any(dim=1).all()
    check_grad("sparse_fp32", g.cpu().numpy(), w, dw.ops01, u)
