"""GPU: the error of the bitflip products and of their gradient against 80-bit
references. An absolute error of S_k = sum log|cos 2 theta_j| is a relative one
of the product, so errors are counted in units of |S_k| 2^-53."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload

pytestmark = pytest.mark.gpu


def _reference(w, C):
    """S_k, the products, and log-derivative factors -2 tan(2 theta_j)."""
    th = 2.0 * w.theta.astype(np.longdouble)
    c = np.cos(th)
    S = (C * np.log(np.abs(c))).sum(axis=1)
    sign = 1.0 - 2.0 * ((C * (c < 0)).sum(axis=1) % 2)
    return S, sign * np.exp(S), -2.0 * np.sin(th) / c


# many gate chunks of few words and few of many; sparse and dense rows of C
@pytest.mark.parametrize("shape", [
    (1000, 100000, 100, (1, 3), (1, 10), 0.4),
    (1000, 60000, 700, (1, 3), (1, 10), 0.4),
    (70, 3000, 200, (1, 30), (1, 30), 0.2),
])
def test_bitflip_error(shape):
    n, m, l, gw, ow, scale = shape
    w = W.small_random(n + m + l, n, m, l, 1, gate_w=gw, op_w=ow, theta_scale=scale)
    dw = DevWorkload(w)
    C = oracle.parity(n, dw.ops01, w.gates)
    S, p, tn = _reference(w, C)
    keep = np.abs(S) > 8.0  # elsewhere the exponential's own rounding counts
    assert keep.sum() > l // 4 and np.abs(S).max() < 700.0
    unit = np.abs(S).astype(np.float64) * 2.0 ** -53
    circ = api.Circuit(n, dw.gens, dw.theta)
    mean = api.iqp_bitflip_expval(circ, dw.ops).cpu().numpy()
    e = (np.abs(mean / p - 1.0).astype(np.float64) / unit)[keep]
    # the last rounding of S_k: uniform within +-ulp / 2 <= |S| 2^-53, 0.58 rms; the rest
    # (cosines, logarithms, short chains) adds less in square
    assert np.sqrt((e * e).mean()) < 0.85
    # gates that one observable alone anticommutes with, one at a time
    u = np.zeros(l)
    pick = np.nonzero(keep)[0][::max(1, keep.sum() // 8)]
    errs = []
    for k in pick:
        u[:] = 0.0
        u[k] = 1.5
        g = api.iqp_bitflip_expval_grad(circ, dw.ops, torch.from_numpy(u).cuda()).cpu().numpy()
        J = np.nonzero(C[k])[0]
        ref = u[k] * p[k] * tn[J]
        errs.append(np.abs((g[J] - ref) / ref).astype(np.float64).mean() / unit[k])
    errs = np.array(errs)
    assert np.sqrt((errs * errs).mean()) < 0.85


def _deep(count):
    """`count` gates of cos(1.5) and one of cos(2 theta) ~ 2e-8 on qubit 0."""
    theta = np.full(count + 1, 0.75)
    theta[count] = np.pi / 4 - 1e-8
    return W.Workload("deep", 2, W.rows_from_lists([[0]] * (count + 1)), theta,
                      W.rows_from_lists([[0], [1]]), np.zeros((1, 2), dtype=np.uint8))


@pytest.mark.parametrize("count", [230, 250, 256, 260])
@pytest.mark.parametrize("u0", [1.0, -1e-6, 1e-12, 1e-18, 1e-24])
def test_bitflip_small_weight_times_small_product(count, u0):
    # u e^S is among the subnormal doubles, or 0, where u e^{S - log|c|} is not
    w = _deep(count)
    dw = DevWorkload(w)
    th = 2.0 * w.theta.astype(np.longdouble)
    c = np.cos(th)
    ref = -2.0 * np.sin(th) * u0 * np.prod(c) / c
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    u = torch.tensor([u0, 3.0], dtype=torch.float64, device="cuda")
    g = api.iqp_bitflip_expval_grad(circ, dw.ops, u).cpu().numpy()
    normal = np.abs(ref) > 1e-306
    # S and log|c_j| are rounded at 700 and under, a few times
    assert (np.abs((g - ref) / ref)[normal] < 1e-12).all()
    assert np.abs(g - ref)[~normal].max(initial=0.0) < 1e-318


def test_bitflip_infinite_weight_of_a_deep_product():
    w = _deep(260)  # S = -706
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    u = torch.tensor([np.inf, 3.0], dtype=torch.float64, device="cuda")
    assert torch.isinf(api.iqp_bitflip_expval_grad(circ, dw.ops, u)).all()
