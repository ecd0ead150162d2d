"""GPU: batches whose parities' blocks, cut to fill the chip for one circuit, are
more than it takes: the same circuit alone and twelve times, bitwise."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2501_04776_amd import BatchPlan, Circuit
from tests.gpu_util import DevWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [60, 500, 1500, 3000, 6000])
def test_batch_blocking_does_not_change_bits(n):
    w = W.small_random(n, n, 9000, 300, 1500, theta_scale=0.3)
    dw = DevWorkload(w)
    problem = (Circuit(n, dw.gens, dw.theta), dw.ops, dw.samples)
    u = torch.from_numpy(np.random.default_rng(1).normal(size=w.l)).cuda()
    out = []
    for count in (1, 12):
        plan = BatchPlan([problem] * count, "split_bf16")
        plan.set_config(fwd_split=0)
        means, ses = plan.expval()
        grads = plan.expval_grad([u] * count)
        out.append((means, ses, plan.phases, grads))
    for one, many in zip(*out):
        assert all(torch.equal(one[0], x) for x in many)
