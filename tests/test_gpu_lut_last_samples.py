"""GPU: the table-lookup gradient where the last chunk of a block holds few samples
or none, phases saved and recomputed, each with one and with two chunks a block: the
samples past s count for nothing."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload, check_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [3, 1280])  # one and, from 1025 samples on, two chunks a block
@pytest.mark.parametrize("s", [1, 3, 5, 1023, 1025, 1027, 2047, 2049, 3073])
def test_last_samples(l, s):
    w = W.small_random(900 + s, 20, 150, l, s, theta_scale=0.3)
    dw = DevWorkload(w)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    u = np.random.default_rng(4).normal(size=l)
    ud = torch.from_numpy(u).cuda()
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, "sparse_fp32", phase_save=True)
    g = api.iqp_expval_grad(circ, dw.ops, dw.samples, ud, ph, "sparse_fp32")
    r = api.iqp_expval_grad(circ, dw.ops, dw.samples, ud, None, "sparse_fp32")
    assert torch.equal(g, r)
    check_grad("sparse_fp32", g.cpu().numpy(), w, dw.ops01, u)
