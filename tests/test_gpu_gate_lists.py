"""GPU: the dense backward over the gate lists of each observable block.
Observables arranged so that every list class occurs: blocks where all gates
are listed, where each half of the block has gates of its own, where one half
is empty, and where nothing is listed; list lengths around the tile sizes and
the segments of the list kernel."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload, check_grad

pytestmark = pytest.mark.gpu


def _workload(m, seed):
    """96 qubits. Rows 0-31 act on qubits 0-15, rows 32-63 on qubits 16-31
    (disjoint gates per half), rows 64-95 on 0-15 and 96-127 on nothing, rows
    128-255 on nothing, rows 256-383 on qubits 32-39 in the first 32 rows only,
    rows 384-447 on anything; gates of weight 1-2 on all qubits, the last
    fifth of them on qubits 40-47, which no row before 384 touches."""
    n, l, s = 96, 448, 200
    rng = np.random.default_rng(seed)
    ops = np.zeros((l, n), dtype=np.uint8)
    for rows, lo, hi in ((range(0, 32), 0, 16), (range(32, 64), 16, 32), (range(64, 96), 0, 16),
                         (range(256, 288), 32, 40), (range(384, 448), 0, 96)):
        for k in rows:
            ops[k, lo + rng.choice(hi - lo, size=rng.integers(1, 4), replace=False)] = 1
    gates = []
    for j in range(m):
        lo, hi = (40, 48) if j >= m - m // 5 else (0, 96)
        gates.append(sorted(lo + rng.choice(hi - lo, size=rng.integers(1, 3), replace=False)))
    theta = rng.uniform(-np.pi, np.pi, size=m)
    return W.Workload("lists", n, W.rows_from_lists(gates), theta, W.dense_to_rows(ops),
                      rng.integers(0, 2, size=(s, n), dtype=np.uint8))


@pytest.mark.parametrize("prec", ["fp32", "split_bf16", "split3_bf16", "split_bf16_fp8"])
@pytest.mark.parametrize("m", [1, 127, 513, 1024, 1025, 2600])
@pytest.mark.parametrize("tile", [None, "2x4", "2x2"])
def test_listed_gates_match_oracle(prec, m, tile, monkeypatch):
    if tile:
        monkeypatch.setenv("IQP_BWD_TILE", tile)
    w = _workload(m, 900 + m)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, prec, phase_save=True)
    for seed, part in ((1, slice(None)), (2, slice(0, 384))):
        u = np.zeros(w.l)
        u[part] = np.random.default_rng(seed).normal(size=len(u[part]))
        g = api.iqp_expval_grad(circ, dw.ops, dw.samples, torch.from_numpy(u).cuda(), ph, prec)
        again = api.iqp_expval_grad(circ, dw.ops, dw.samples, torch.from_numpy(u).cuda(), ph, prec)
        torch.cuda.synchronize()
        g = g.cpu().numpy()
        # the lists' order varies from run to run, the gradient does not
        assert np.array_equal(g, again.cpu().numpy())
        check_grad(prec, g, w, dw.ops01, u)
    # gates that commute with every weighted observable
    C = oracle.parity(w.n, dw.ops01[:384], w.gates)
    assert (g[C.sum(axis=0) == 0] == 0.0).all()


@pytest.mark.parametrize("prec", ["split_bf16", "split3_bf16", "split_bf16_fp8"])
def test_no_listed_gate(prec):
    # observables of weight 0 only: every list is empty
    w = _workload(300, 5)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    ops = dw.ops[128:256].contiguous()
    u = torch.ones(128, dtype=torch.float64, device="cuda")
    g = api.iqp_expval_grad(circ, ops, dw.samples, u, None, prec)
    assert (g == 0.0).all()
