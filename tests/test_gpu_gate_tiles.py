"""GPU: the split-BF16 backward whose lists are split by the halves of a block,
where its tiles hold one class each and where they hold all classes together,
bitwise against the wave tile whose lists are not split."""
import numpy as np
import pytest
import torch

from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload
from tests.test_gpu_gate_lists import _workload

pytestmark = pytest.mark.gpu


# one tile holds 512 gates; the blocks of _workload list a half, both, or none
@pytest.mark.parametrize("m", [3, 300, 512, 700, 1500, 2600, 5200])
def test_tiles_of_all_classes_bitwise(m, monkeypatch):
    monkeypatch.setenv("IQP_BWD_SPLITS", "1")
    w = _workload(m, 40 + m)
    dw = DevWorkload(w)
    circ = api.Circuit(w.n, dw.gens, dw.theta)
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, "split_bf16", phase_save=True)
    u = torch.from_numpy(np.random.default_rng(6).normal(size=w.l)).cuda()
    got = {}
    for tile in ("2x2", "2x4"):
        monkeypatch.setenv("IQP_BWD_TILE", tile)
        got[tile] = api.iqp_expval_grad(circ, dw.ops, dw.samples, u, ph, "split_bf16")
    assert torch.equal(got["2x2"], got["2x4"])
