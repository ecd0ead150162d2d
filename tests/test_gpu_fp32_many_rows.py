"""GPU: the FP32 gradient from saved phases at the most observables a call takes,
2^24, one more than a grid has blocks."""
import numpy as np
import pytest
import torch

from paper_2501_04776_amd import api

pytestmark = pytest.mark.gpu


def test_fp32_gradient_of_2_24_observables():
    n, m, l = 10, 128, 1 << 24
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    gens = torch.randint(1, 1 << n, (m, 1), generator=g, device="cuda")
    # weight 0 for most: C is sparse
    ops = torch.randint(0, 1 << n, (l, 1), generator=g, device="cuda")
    ops[torch.rand(l, generator=g, device="cuda") < 0.9] = 0
    z = torch.randint(0, 1 << n, (1, 1), generator=g, device="cuda")
    ph = (torch.rand((l, 1), generator=g, device="cuda") - 0.5) * 6.0
    u = torch.randn(l, generator=g, device="cuda", dtype=torch.float64)
    theta = torch.zeros(m, dtype=torch.float64, device="cuda")
    got = api.iqp_expval_grad(api.Circuit(n, gens, theta), ops, z, u, ph, "fp32").cpu().numpy()
    # the observables by their bits, then dtheta_j = -2 b_j sum_k c_kj u_k sin(phase_k)
    w = u * torch.sin(ph[:, 0].to(torch.float64))
    by_bits = torch.bincount(ops[:, 0], weights=w, minlength=1 << n).cpu().numpy()
    gv, zv = gens[:, 0].cpu().numpy(), int(z[0, 0])
    odd = np.array([[bin(v & j).count("1") & 1 for v in range(1 << n)] for j in gv])
    b = np.array([1.0 - 2.0 * (bin(zv & j).count("1") & 1) for j in gv])
    ref = -2.0 * b * (odd * by_bits).sum(axis=1)
    # weights and sums of up to 64 rows in FP32: at most 64 roundings of 2^-24 each
    scale = 2.0 * (odd * torch.bincount(ops[:, 0], weights=w.abs(),
                                        minlength=1 << n).cpu().numpy()).sum(axis=1)
    assert (np.abs(got - ref) <= 64 * 2.0 ** -24 * scale).all()
