"""GPU: the bitflip products where their blocks take fewer row words than fit
(few observables, and few gates beside many), against sums of logarithms."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload

pytestmark = pytest.mark.gpu

RTOL = 1e-11


# row words per block by the rows there are and by a block per CU, on both sides
# of each halving; gate chunks fewer, as many and more than the threads over them
@pytest.mark.parametrize("n", [10, 500, 1100, 2000])
@pytest.mark.parametrize("shape", [(50, 1000), (300, 129), (2000, 257), (4096, 70), (4200, 640),
                                   (33000, 20), (12000, 1500)])
def test_bitflip_few_blocks(n, shape):
    m, l = shape
    w = W.small_random(n + m + l, n, m, l, 1, gate_w=(1, 3), op_w=(1, 4), theta_scale=0.2)
    dw = DevWorkload(w)
    circ = api.Circuit(n, dw.gens, dw.theta)
    u = np.random.default_rng(3).normal(size=l)
    mean = api.iqp_bitflip_expval(circ, dw.ops).cpu().numpy()
    g = api.iqp_bitflip_expval_grad(circ, dw.ops, torch.from_numpy(u).cuda()).cpu().numpy()
    # all cosines are positive
    C = oracle.parity(n, dw.ops01, w.gates).astype(np.float64)
    rm = np.exp(C @ np.log(np.cos(2.0 * w.theta)))
    rg = -2.0 * np.tan(2.0 * w.theta) * (C.T @ (u * rm))
    assert np.allclose(mean, rm, rtol=RTOL, atol=0.0)
    assert np.allclose(g, rg, rtol=1e-10, atol=1e-12 * np.abs(rg).max())
