"""GPU: the FP32 gradient over the non-zero entries of C where a row ends on a
list: no entry, one list of 1024 and two, and one entry more or less, bitwise
against the batched form, which always takes the matrix cores."""
import numpy as np
import torch
import pytest

import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload

pytestmark = pytest.mark.gpu


def test_fp32_gradient_rows_of_whole_lists(monkeypatch):
    # gates on single qubits: observable {q} anticommutes with the gates on q
    counts = [1023, 1024, 1025, 2047, 2048, 2049, 1]
    n, m, s = 400, 30000, 2100
    rng = np.random.default_rng(31)
    q = rng.permutation(np.concatenate([np.repeat(np.arange(len(counts)), counts),
                                        rng.integers(len(counts), n, m - sum(counts))]))
    ops = [[]] + [[k] for k in range(len(counts))] + [[]] * 100
    ops += [[k] for k in rng.integers(len(counts), n, 100)]
    w = W.Workload("row ends", n, W.rows_from_lists([[int(x)] for x in q]),
                   rng.uniform(-np.pi, np.pi, m), W.rows_from_lists(ops),
                   W.uniform_bits(rng, s, n))
    assert w.l * s * m >= 2 ** 31
    monkeypatch.setenv("IQP_BWD_SPLITS", "1")
    dw = DevWorkload(w)
    circ = api.Circuit(n, dw.gens, dw.theta)
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, "fp32", phase_save=True)
    u = torch.from_numpy(rng.normal(size=w.l)).cuda()
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, u, ph, "fp32")
    plan = api.BatchPlan([(circ, dw.ops, dw.samples)], "fp32")
    plan.phases[0].copy_(ph)
    (ref,) = plan.expval_grad([u])
    assert torch.equal(g, ref)
