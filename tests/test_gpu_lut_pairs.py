"""GPU: the table-lookup gradient with two chunks of 1024 samples a block (even
chunks: from 640 such blocks on, odd: 1280; shared samples), at the lines and at
the edges of a chunk and of a pair, also where a bounded grid strides over its
units; independent sets and single chunks around the same sizes."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload, check_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,s,cap,indep", [
    (639, 1500, 0, False), (640, 1025, 0, False), (640, 2048, 7, False), (641, 1024, 0, False),
    (320, 3073, 0, False), (320, 4096, 7, False), (639, 2049, 0, False), (640, 2049, 0, False),
    (640, 3072, 7, False), (427, 4097, 0, False), (640, 1500, 0, True), (1300, 700, 0, True)])
def test_pairs_of_chunks(l, s, cap, indep, monkeypatch):
    if cap:
        monkeypatch.setenv("IQP_SPARSE_GRID_CAP", str(cap))
    # some rows of C hold more than one list of 1024 generators
    w = W.small_random(700 + s, 30, 2500 if s < 2000 else 200, l, s, theta_scale=0.2)
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
