"""GPU: the table-lookup forward's exchange of parity words over a wave. Phases
of single samples show which sample came to which lane and which generator to
which table, at the edges of words (32, 64), waves (256) and chunks (1024) of
samples and of groups (64), tables (4) and lists (1024) of generators."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import TOL, DevWorkload, check_grad, wrap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("indep", [False, True])
@pytest.mark.parametrize("s,m", [(1, 3), (33, 130), (65, 127), (257, 1), (1023, 515), (1025, 64),
                                 (2049, 700), (300, 4500)])
def test_phases(s, m, indep):
    l = 6
    w = W.small_random(100 + s, 40, m, l, s, theta_scale=0.2)
    dw = DevWorkload(w)
    circ = api.Circuit(dw.n, dw.gens, dw.theta)
    om, ose, oph = oracle.expval(w.n, w.gates, w.theta, dw.ops01, w.samples, phases=True)
    u = np.random.default_rng(1).normal(size=l)
    ud = torch.from_numpy(u).cuda()
    if indep:
        z = dw.samples.expand(l, *dw.samples.shape).contiguous()
        mean, se, ph = api.iqp_expval_indep(circ, dw.ops, z, phase_save=True)
        g = api.iqp_expval_indep_grad(circ, dw.ops, z, ud, ph)
    else:
        mean, se, ph = api.iqp_expval(circ, dw.ops, dw.samples, "sparse_fp32", phase_save=True)
        g = api.iqp_expval_grad(circ, dw.ops, dw.samples, ud, ph, "sparse_fp32")
    assert np.abs(mean.cpu().numpy() - om).max() < TOL["sparse_fp32"]
    # rounding: each angle once (in T and in the sum, which counts twice), 32 of
    # them in a tree of 7 adds, then a fold of 3 operations below pi plus the
    # tree's sum (its whole counts times the float pi are exact in 64 bits); the
    # phase itself
    t = 2.0 * np.abs(w.theta).max()
    groups = -(-m // 32)
    tol = 2.0 ** -24 * (3 * m * t + 2 * groups * (7 * 32 * t + 3 * (np.pi + 32 * t)) + 2 * np.pi)
    assert np.abs(wrap(ph.cpu().numpy() - oph)).max() < tol
    check_grad("sparse_fp32", g.cpu().numpy(), w, dw.ops01, u)
