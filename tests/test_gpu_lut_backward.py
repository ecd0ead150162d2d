"""GPU: the table-lookup gradient with two chunks of 1024 samples a block (from
320 such blocks on), at the edges of a chunk and of a pair, also where a bounded
grid strides over its units; 319 blocks take one chunk each."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload, check_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("indep", [False, True])
@pytest.mark.parametrize("l,s,cap", [(319, 700, 0), (320, 1, 0), (320, 1024, 7), (161, 2049, 0),
                                     (321, 1025, 0), (160, 3072, 7), (110, 4097, 0)])
def test_pairs_of_chunks(l, s, cap, indep, monkeypatch):
    if cap:
        monkeypatch.setenv("IQP_SPARSE_GRID_CAP", str(cap))
    # some rows of C hold more than one list of 1024 generators
    w = W.small_random(300 + s, 30, 2500 if s < 2000 else 200, l, s, theta_scale=0.2)
    dw = DevWorkload(w)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    u = np.random.default_rng(2).normal(size=l)
    ud = torch.from_numpy(u).cuda()
    if indep:
        z = dw.samples.expand(l, *dw.samples.shape).contiguous()
        g = api.iqp_expval_indep_grad(circ, dw.ops, z, ud)
    else:
        g = api.iqp_expval_grad(circ, dw.ops, dw.samples, ud, precision="sparse_fp32")
    check_grad("sparse_fp32", g.cpu().numpy(), w, dw.ops01, u)
