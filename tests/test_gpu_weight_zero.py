"""GPU: observables of weight 0 among others. The MMD forward leaves their rows
out of the dense product, and the sparse kernels skip their rows of C; nothing
of the others may change, and the weight-0 ones stay exact."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import TOL, DevWorkload, check_grad

pytestmark = pytest.mark.gpu


def _workload(l, keep, s=1300, m=9000, n=70, seed=21):
    """l observables, those of weight > 0 given by the mask `keep`."""
    w = W.small_random(seed, n, m, l, s, theta_scale=0.2, with_data=50)
    ops = W.rows_to_dense(w.ops, n)
    ops[~keep] = 0
    w.ops = W.dense_to_rows(ops)
    return w


# the dense forward leaves rows out from 2^34 terms on
@pytest.mark.parametrize("prec", ["split_bf16", "split3_bf16", "split_bf16_fp8"])
@pytest.mark.parametrize("kind", ["none", "all but one", "most", "whole tiles", "all"])
def test_mmd_matches_smaller_calls(prec, kind):
    l = 1500
    rng = np.random.default_rng(4)
    keep = {"none": np.ones(l, bool), "all but one": np.arange(l) == 777,
            "most": rng.random(l) < 0.2, "whole tiles": np.arange(l) >= 1024,
            "all": np.zeros(l, bool)}[kind]
    w = _workload(l, keep)
    assert w.l * w.s * w.m >= 2 ** 34
    dw = DevWorkload(w)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    wt = torch.from_numpy(rng.random(l)).cuda()
    loss, g = api.iqp_mmd_loss_grad(circ, dw.ops, wt, dw.samples, dw.data, True, True, prec)
    # the same operators in calls below the line, 128 rows (two gradient blocks
    # of every form) at a time
    ref, gref = 0.0, torch.zeros_like(g)
    for a in range(0, l, 128):
        x, y = api.iqp_mmd_loss_grad(circ, dw.ops[a:a + 128].contiguous(), wt[a:a + 128],
                                     dw.samples, dw.data, True, True, prec)
        ref, gref = ref + x.item(), gref + y
    scale = max(1.0, float(gref.abs().max()))
    # FP32 partial sums are split over the samples differently
    assert abs(loss.item() - ref) < 1e-9 * max(1.0, abs(ref))
    assert float((g - gref).abs().max()) < 1e-6 * scale


@pytest.mark.parametrize("indep", [False, True])
def test_sparse_skips_weight_zero(indep):
    keep = np.arange(70) % 3 != 0
    w = _workload(70, keep, s=1100, m=1500, seed=5)
    dw = DevWorkload(w)
    ops01 = W.rows_to_dense(w.ops, w.n)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    u = np.random.default_rng(1).normal(size=w.l)
    ud = torch.from_numpy(u).cuda()
    if indep:
        z = dw.samples.expand(w.l, *dw.samples.shape).contiguous()
        mean, se, ph = api.iqp_expval_indep(circ, dw.ops, z, phase_save=True)
        g = api.iqp_expval_indep_grad(circ, dw.ops, z, ud, ph)
    else:
        mean, se, ph = api.iqp_expval(circ, dw.ops, dw.samples, "sparse_fp32", phase_save=True)
        g = api.iqp_expval_grad(circ, dw.ops, dw.samples, ud, ph, "sparse_fp32")
    om, ose = oracle.expval(w.n, w.gates, w.theta, ops01, w.samples)
    assert np.abs(mean.cpu().numpy() - om).max() < TOL["sparse_fp32"]
    zero = torch.from_numpy(~keep).cuda()
    assert (mean[zero] == 1.0).all() and (se[zero] == 0.0).all() and (ph[zero] == 0.0).all()
    check_grad("sparse_fp32", g.cpu().numpy(), w, ops01, u)
