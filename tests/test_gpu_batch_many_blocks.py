"""GPU: a batch of so many circuits that their parities, cut into the blocks that
one circuit alone takes (64 rows of 64 words and more, 256 gates), would take
more of them than one grid holds."""
import pytest
import torch

from paper_2501_04776_amd import BatchPlan, Circuit

pytestmark = pytest.mark.gpu


def test_batch_of_2_24_parity_blocks():
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GiB of free GPU memory")
    # two row words and 384 groups of 256 gates for each of C and B
    n, m, rows = 4096, 98304, 128
    count = (1 << 24) // (2 * 2 * 384) + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    gens = torch.zeros((m, n // 64), dtype=torch.int64, device="cuda")
    for _ in range(3):
        q = torch.randint(0, n, (m,), generator=g, device="cuda")
        gens[torch.arange(m, device="cuda"), q // 64] |= torch.ones_like(q) << (q % 64)
    theta = torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * 0.02
    bits = (2, rows, n // 64)
    ops, z = torch.randint(-2 ** 63, 2 ** 63 - 1, bits, generator=g, device="cuda")
    problem = (Circuit(n, gens, theta), ops.contiguous(), z.contiguous())
    # the gate-word splits of a pass follow from all its problems: none here
    one = BatchPlan([problem], "split_bf16", graph=False, save_phases=False)
    plan = BatchPlan([problem] * count, "split_bf16", graph=False, save_phases=False)
    for p in (one, plan):
        p.set_config(fwd_split=0)
    ref, _ = one.expval()
    plan.ws.fill_(255)
    means, _ = plan.expval()
    same = torch.stack([(x == ref[0]).all() for x in means])
    assert bool(same.all()), same.logical_not().nonzero().flatten()[:8].tolist()
    del plan, means
    torch.cuda.empty_cache()
